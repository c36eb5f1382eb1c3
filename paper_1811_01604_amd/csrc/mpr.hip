// MI355X (gfx950) implementation of the C ABI in include/mpr.h: MPR gap
// filling with the checkerboard hybrid Monte Carlo sweep (arXiv:1811.01604,
// Algorithms 1 and 2, Section 3.3).
//
// Kernels
//   init_chains       gap angles U(0, 2 pi) from Philox (Algorithm 2 step 2.2)
//                     or a warm start; samples stored with the sign bit set
//   half_sweep        Algorithm 1 on the gap sites of one colour for every
//                     chain; the colour-1 pass also sums all bond energies
//                     (every bond has exactly one colour-1 end) and both
//                     passes count accepted proposals
//   control           Algorithm 2 steps 5.2-5.5 and 6 per chain: a-rule,
//                     e(i+1), Savitzky-Golay slope, phase changes
//   finalize          sum of the M states per gap site
//   map_*, predict    equation (map) and its inverse
//   sample_energy     equation (mpr-sse)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <map>
#include <mutex>
#include <string>
#include <type_traits>
#include <tuple>
#include <utility>
#include <vector>

#include "../../include/mpr.h"
#include "mpr_device.h"

static_assert(sizeof(mpr_params) == 128, "mpr_params layout");

using namespace mpr;

namespace {

constexpr int kBlock = 256;
constexpr int kMapBlocks = 512;          // partial-result blocks per image at most (map, e_s)
constexpr int kHoldoutBlocks = 64;       // partial-result blocks of the hold-out error
constexpr size_t kScratchBytes = 8u << 20;
constexpr size_t kHaloBytes = 8u << 20;  // halo words of the resident sweeps, after the scratch
constexpr uint32_t kTableStream = 0x80000000u;
constexpr uint32_t kInitSweep = 0xFFFFFFFFu;
// Layout of the context's device scratch: fixed slots, then a region for
// per-call partial results.
constexpr int64_t kDoneOffset = 0;       // done-chain counter
constexpr int64_t kTicketOffset = 256;   // last-block ticket of the redo kernel with the control fused
constexpr int64_t kGenOffset = 512;      // four words of a resident launch (kResArrive, kResGoes, kResStart)
constexpr int64_t kAbortOffset = 768;    // time-out word of the resident sweeps
constexpr int64_t kSlotsOffset = 16384;  // the blocks' sums of the resident sweeps
constexpr int64_t kWorkOffset = 1024;    // three work counters (profiling)
constexpr int64_t kEnergyOffset = 2048;  // diag energy accumulator
constexpr int64_t kSlopeOffset = 4096;   // diag slope input / output
constexpr int64_t kVarOffset = 65536;    // per-call partials
constexpr int64_t kHostWordsBytes = 1024;      // pinned mirror of the control words
constexpr int64_t kHostStageBytes = 64 << 10;  // pinned host block (control words + staging)
static_assert(kAbortOffset + 4 <= kHostWordsBytes && kGenOffset + 4 <= kHostWordsBytes,
              "the control words are read back in one copy");
constexpr int kCompactSites = 4 * kBlock;  // sites per block of the compacted sweep shapes
constexpr int kRecordSegs = 32;            // blocks per chain of record_states_kernel
constexpr int kWarmMinStates = 100;        // default of mpr_params.warm_min_states

// Workspace of mpr_simulate_noalloc, for callers that cannot allocate: one
// copy per device, held by the library's code object until the process
// ends.  Host code never passes the array's name to a kernel (on the host it
// is a stand-in, not a device address); it uses the address that
// hipGetSymbolAddress returns on each device, kept per device by static_ws_addr.
constexpr int64_t kStaticWorkspaceBytes = (int64_t)64 << 20;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char static_workspace[kStaticWorkspaceBytes];

// Sites whose single-precision decision is too close to call are not written
// by the sweep kernels: they set the site's bit in their block's mask (one
// bit per site of the block, site = 2 pair + slot) and the block's bit in a
// bitmap, and redo_fp64_kernel redoes them in double precision afterwards.
// Keeping the double-precision code out of the sweep kernels keeps them at
// fewer than 64 registers.
struct Redo {
    uint32_t *mask;    // words_per_block per sweep block (flattened block index)
    uint32_t *blocks;  // one bit per sweep block
};

__device__ __forceinline__ void defer_redo(const Redo &rd, uint32_t gb, int words, uint32_t idx)
{
    atomicOr(&rd.mask[(size_t)gb * words + (idx >> 5)], 1u << (idx & 31u));
    atomicOr(&rd.blocks[gb >> 5], 1u << (gb & 31u));
}

// Parameters of the control kernel.
struct CtlParams {
    double a_targ, k_a, q;
    double e_unit;        // energy fixed-point unit of the sweep kernels
    int32_t angle_bytes;  // bytes per stored angle (4 or 8), for the work counters
    int32_t n_f, n_fit, i_max, fixed_relax, eq_a_mode, K, burn, meas;
    double w[kMaxFit];  // Savitzky-Golay derivative weights, oldest first
};

struct ImgDev {
    int64_t offset;
    int32_t nx, ny;
};

// The images of a call and their data ranges.  A few of them travel in the
// kernel's arguments (a copy to the device before the launch costs some 8 us
// of a small call), more in device memory.
constexpr int kArgImages = 8;
struct ImgArgs {
    const ImgDev *dev;  // null: own
    ImgDev own[kArgImages];
    // (uniform over the wave: b is a block index)
    __device__ ImgDev at(int b) const
    {
        ImgDev r = dev ? dev[b] : own[b];
        r.offset = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(r.offset >> 32)) << 32) |
                             (uint32_t)__builtin_amdgcn_readfirstlane((int)r.offset));
        r.nx = __builtin_amdgcn_readfirstlane(r.nx);
        r.ny = __builtin_amdgcn_readfirstlane(r.ny);
        return r;
    }
};
struct RangeArgs {
    const double *dev;  // null: own
    double own[2 * kArgImages];
    __device__ double lo(int b) const { return dev ? dev[2 * b] : own[2 * b]; }
    __device__ double hi(int b) const { return dev ? dev[2 * b + 1] : own[2 * b + 1]; }
};
constexpr int kMaxProbs = 64;
struct ProbArgs {
    double v[kMaxProbs];
};

// Head of a simulate workspace: what a resumed call checks before it
// continues the run the workspace holds.
struct RunHeader {
    uint64_t magic;     // kRunMagic
    uint64_t key;       // run_key of the images and parameters
    int64_t bytes;      // sim_bytes of the run
    int32_t n_chains;
    int32_t state;      // 1: stopped at sweep_limit with chains running (resumable)
};

}  // namespace

// ====================================================================== kernels

// Slope of the energy series from the ring buffer: sum_j w_j e(t+1-n_fit+j).
__device__ double ring_slope(const double *ring, uint32_t t, int n_fit, const double *w)
{
    double s = 0.0;
    for (int j = 0; j < n_fit; ++j) {
        // e(t + 1 - n_fit + j) was stored at slot (t + 1 - n_fit + j) mod n_fit
        const uint32_t idx = (t + 1u + (uint32_t)j) % (uint32_t)n_fit;
        s += w[j] * ring[idx];
    }
    return s;
}

// (fp64: the chains hold doubles; a gap starts at 2 pi u in double, as in
// the plain definition.)  Every word of the half-grids is written, zeros in
// the padding beyond a row's sites: a thread takes four half-columns of one
// row and colour, so that its stores are whole 16-byte groups and no memset
// goes before (two or four per chain: 768 of them took 3 ms of a 24-image,
// 192-chain batch).  Bound by those writes; 4096^2, 16 chains: 927 us before,
// 790 us now.
template <typename RT>
__global__ __launch_bounds__(kBlock) void init_chains_kernel(const ChainDesc *__restrict__ descs,
                                                             const int64_t *__restrict__ offsets,
                                                             const float *__restrict__ phi,
                                                             const uint8_t *__restrict__ sampled,
                                                             const float *__restrict__ phi_init, uint32_t seed_lo,
                                                             uint32_t seed_hi, int table_mode, RunHeader hdr,
                                                             RunHeader *__restrict__ d_hdr)
{
    if (d_hdr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *d_hdr = hdr;
    typedef RT v4 __attribute__((ext_vector_type(4)));
    const ChainDesc d = descs[blockIdx.y];
    const int64_t off = offsets[blockIdx.y];
    const uint32_t nq = (uint32_t)d.S >> 2;
    const int64_t n = (int64_t)d.ny * nq * 2;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        // the two colours of a row one after the other, groups along the row
        const uint32_t yc = (uint32_t)(i / nq);
        const int q = (int)(i - (int64_t)yc * nq), y = (int)(yc >> 1), c = (int)(yc & 1u);
        const int s = (y + c) & 1;
        v4 out = {(RT)0, (RT)0, (RT)0, (RT)0};
        U4 w = {0u, 0u, 0u, 0u};
        for (int e = 0; e < 4; ++e) {
            const int x = 2 * (4 * q + e) + s;
            // two neighbouring sites of a colour share one Philox call
            if (!table_mode && !phi_init && (e & 1) == 0) {
                const U4 ctr = {(uint32_t)y * (uint32_t)d.nx + ((uint32_t)x & ~2u), kInitSweep, d.chain, d.image_id};
                w = philox4x32_10(ctr, seed_lo, seed_hi);
            }
            if (x >= d.nx) continue;
            const int64_t j = off + (int64_t)y * d.nx + x;
            double v;
            bool fixed = false;
            if (table_mode) {
                v = kPi;
            } else if (sampled[j]) {
                v = (double)fabsf(phi[j]);
                fixed = true;
            } else if (phi_init) {
                // a given start is reduced into [0, 2 pi) with its sign bit clear
                // (a set sign bit marks a sampled site; -0.0 included)
                v = (double)phi_init[j];
                if (!(v >= 0.0 && v < kTwoPi)) {
                    v -= kTwoPi * floor(v / kTwoPi);
                    if (!(v >= 0.0 && v < kTwoPi)) v = 0.0;
                }
                v = fabs(v);
                if (sizeof(RT) == 4 && (float)v >= 6.28318548f) v = 6.28318501;  // the largest float below 2 pi
            } else {
                v = kTwoPi * (double)unit24((e & 1) ? w.z : w.x);
            }
            if constexpr (sizeof(RT) == 8) out[e] = fixed ? mark_fixed_d(v) : v;
            else out[e] = fixed ? mark_fixed((float)v) : (float)v;
        }
        const int64_t j = (int64_t)y * d.S + 4 * q;
        const v4 zero = {(RT)0, (RT)0, (RT)0, (RT)0};
        // select by value: indexing the descriptor with c would put it in memory
        *(v4 *)((RT *)(c ? d.h[1] : d.h[0]) + j) = out;
        RT *h2 = (RT *)(c ? d.h2[1] : d.h2[0]), *ap = (RT *)(c ? d.acc[1] : d.acc[0]), *mp = (RT *)(c ? d.m2[1] : d.m2[0]);
        if (h2) *(v4 *)(h2 + j) = out;
        if (ap) *(v4 *)(ap + j) = zero;
        if (mp) *(v4 *)(mp + j) = zero;
    }
}

// A full row-major grid of double angles (gaps: the starting state) into the
// half-grids of one double-precision chain, samples marked.
__global__ void split_fp64_kernel(const ChainDesc *__restrict__ descs, const double *__restrict__ phi,
                                  const uint8_t *__restrict__ sampled)
{
    const ChainDesc d = descs[0];
    const int64_t n = (int64_t)d.nx * d.ny;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int y = (int)(i / d.nx);
        const int x = (int)(i - (int64_t)y * d.nx);
        const double v = fabs(phi[i]);
        double *hp = (double *)(((x + y) & 1) ? d.h[1] : d.h[0]);
        hp[(int64_t)y * d.S + (x >> 1)] = sampled[i] ? mark_fixed_d(v) : v;
    }
}

// Chain of a flattened block index: start[c] <= b < start[c + 1].  The
// search runs on block-uniform values, so it stays in scalar registers.
__device__ __forceinline__ int find_chain(const int64_t *__restrict__ start, int n, int64_t b)
{
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (start[mid] <= b) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The blocks of a sweep launch, laid end to end over the chains it covers
// (the chains not yet done): launch chain k < n owns blocks start[k] <= b <
// start[k + 1] and is chain id[k] of the chain set.
struct BlockMap {
    const int64_t *start;
    const int32_t *id;
    int32_t n;
    int32_t pad;
};

// Chain of block b, and the block's index within that chain.
__device__ __forceinline__ int chain_of_block(const BlockMap &bm, int64_t b, int *local)
{
    const int k = find_chain(bm.start, bm.n, b);
    *local = (int)(b - bm.start[k]);
    return bm.id[k];
}

// Half-sweep of colour `colour` for every chain of a (possibly ragged)
// batch in one launch.  The blocks of all chains are laid end to end
// (start[] = prefix sums of blocks per chain).  A 256-thread block covers
// ROWS half-rows x (256 / ROWS) site pairs; each thread takes the two
// neighbouring sites h0 = 2k and h0 + 1 of one half-row, which share one
// Philox call.  Results do not depend on ROWS: random numbers are keyed by
// site and energies are summed in fixed point.
template <bool DIAG, int ROWS>
__device__ __forceinline__ void half_sweep_body(const ChainDesc *__restrict__ descs,
                                                ChainState *__restrict__ states,
                                                BlockMap bm, int colour,
                                                SweepConsts sc, int or_only, Redo rd, uint8_t *__restrict__ flags)
{
    constexpr int PX = kBlock / ROWS;
    int lb;
    const int c = chain_of_block(bm, (int64_t)blockIdx.x, &lb);
    ChainState *stp = states + c;
    const int phase = stp->phase;
    if (phase == PH_DONE) return;
    const ChainDesc d = descs[c];
    const int nbx = ((d.S >> 1) + PX - 1) / PX;
    const int by = lb / nbx;
    const int bx = lb - by * nbx;
    const int y = by * ROWS + (int)(threadIdx.x / PX);
    const int h0 = 2 * (bx * PX + (int)(threadIdx.x % PX));
    const uint32_t sweep = stp->sweep;
    const float inv_T = stp->inv_T, dscale = stp->dscale;
    const bool want_energy = (colour == 1) && (phase != PH_EQ);
    const bool want_acc = phase != PH_EQ;
    uint32_t e_thread = 0u, acc_thread = 0u;

    if (y < d.ny) {
        const int s = (y + colour) & 1;
        const int W = (d.nx - s + 1) >> 1;
        const int Wo = (d.nx + s) >> 1;
        if (h0 < W) {
            const bool two = (h0 + 1) < W;
            // select by value: indexing d.h with a runtime colour would put
            // the descriptor in memory
            float *mine = colour ? d.h[1] : d.h[0];
            const float *oth = colour ? d.h[0] : d.h[1];
            const int row = y * d.S;
            const bool vL = h0 + s - 1 >= 0, vM = h0 + s < Wo, vR = h0 + s + 1 < Wo;
            const bool vU = y > 0, vD = y + 1 < d.ny;
            // every load is issued, from a clamped in-row position when the
            // neighbour is missing (update_site ignores it by its valid bit),
            // so that all of them are in flight at once
            const float2 v = gldi2(mine, (uint32_t)(row + h0));
            const float oL = angle_of(gldi(oth, (uint32_t)(row + max(h0 + s - 1, 0))));
            const float oM = angle_of(gldi(oth, (uint32_t)(row + h0 + s)));  // h0 + s <= S - 1
            const float oR = angle_of(gldi(oth, (uint32_t)(row + min(h0 + s + 1, d.S - 1))));
            float2 up = gldi2(oth, (uint32_t)(row + (vU ? -d.S : 0) + h0));
            float2 dn = gldi2(oth, (uint32_t)(row + (vD ? d.S : 0) + h0));
            up.x = angle_of(up.x);
            up.y = angle_of(up.y);
            dn.x = angle_of(dn.x);
            dn.y = angle_of(dn.y);
            const bool fixed0 = is_fixed(v.x), fixed1 = !two || is_fixed(v.y);
            const float a0 = angle_of(v.x), a1 = angle_of(v.y);
            float u0 = 0.5f, r0 = 0.5f, u1 = 0.5f, r1 = 0.5f;
            if (!or_only && (!fixed0 || !fixed1)) {
                const U4 ctr = {(uint32_t)y * (uint32_t)d.nx + (uint32_t)(2 * h0 + s), sweep, d.chain, d.image_id};
                const U4 w = philox4x32_10(ctr, sc.seed_lo, sc.seed_hi);
                u0 = unit24(w.x);
                r0 = unit24(w.y);
                u1 = unit24(w.z);
                r1 = unit24(w.w);
            }
            // site h0: left oL, right oM, up, down; site h0 + 1: left oM, right oR
            const uint32_t val0 = (vL ? 1u : 0u) | (vM ? 2u : 0u) | (vU ? 4u : 0u) | (vD ? 8u : 0u);
            const uint32_t val1 = 1u | (vR ? 2u : 0u) | (vU ? 4u : 0u) | (vD ? 8u : 0u);
            bool n0 = true, n1 = true;
            SiteOut o0 = update_site(a0, oL, oM, up.x, dn.x, val0, u0, r0, inv_T, dscale, or_only != 0, &n0);
            SiteOut o1 = update_site(a1, oM, oR, up.y, dn.y, val1, u1, r1, inv_T, dscale, or_only != 0, &n1);
            // too close to call: left unchanged here, redone in double precision
            n0 = n0 && !fixed0;
            n1 = n1 && !fixed1;
            if (n0) defer_redo(rd, blockIdx.x, 2 * kBlock / 32, 2u * threadIdx.x);
            if (n1) defer_redo(rd, blockIdx.x, 2 * kBlock / 32, 2u * threadIdx.x + 1u);
            const bool w0 = !fixed0 && !n0, w1 = two && !fixed1 && !n1;  // sites written here
            const float out0 = w0 ? o0.phi : v.x;
            const float out1 = w1 ? o1.phi : v.y;
            if (two) {
                v2f w;
                w.x = out0;
                w.y = out1;
                *(gv2f *)gaddr(mine, (uint32_t)(row + h0)) = w;
            } else if (w0) {
                gsti(mine, (uint32_t)(row + h0), out0);
            }
            float *accp = colour ? d.acc[1] : d.acc[0];
            if (phase == PH_EQ && accp) {
                float *m2p = colour ? d.m2[1] : d.m2[0];
                const float ik = stp->inv_k, ikm1 = stp->inv_km1;
                if (w0) accumulate_state_i(accp, m2p, (uint32_t)(row + h0), out0, ik, ikm1);
                if (w1) accumulate_state_i(accp, m2p, (uint32_t)(row + h0 + 1), out1, ik, ikm1);
            }
            acc_thread = (w0 && o0.accepted ? 1u : 0u) + (w1 && o1.accepted ? 1u : 0u);
            // a sampled site's bonds are unchanged by this half-sweep
            if (want_energy)
                e_thread = (fixed0 ? energy_fx(o0.e_before) : (w0 ? energy_fx(o0.e_bonds) : 0u)) +
                           (!two ? 0u : fixed1 ? energy_fx(o1.e_before) : (w1 ? energy_fx(o1.e_bonds) : 0u));
            if (DIAG && flags) {
                const int64_t x0 = 2 * h0 + s;
                if (w0) flags[(int64_t)y * d.nx + x0] = (uint8_t)o0.flags;
                if (w1) flags[(int64_t)y * d.nx + x0 + 2] = (uint8_t)o1.flags;
            }
        }
    }
    if (!want_acc) return;
    // Block sums of the energy (split in 16-bit halves so that 32-bit lane
    // sums cannot overflow) and of the accepted count (packed in the top byte).
    uint32_t lo = (e_thread & 0xFFFFu) | (acc_thread << 24);
    uint32_t hi = e_thread >> 16;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo += __shfl_xor(lo, off);
        hi += __shfl_xor(hi, off);
    }
    __shared__ uint32_t red[2][kBlock / 64];
    const int wid = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[0][wid] = lo;
        red[1][wid] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long e = 0ull, a = 0ull;
        for (int i = 0; i < kBlock / 64; ++i) {
            e += ((unsigned long long)red[1][i] << 16) + (red[0][i] & 0xFFFFFFu);
            a += red[0][i] >> 24;
        }
        if (e) atomicAdd(&stp->e_fx, e);
        if (a) atomicAdd(&stp->acc, a);
    }
}

template <bool DIAG, int ROWS>
__global__ __launch_bounds__(kBlock) void half_sweep_kernel(const ChainDesc *__restrict__ descs,
                                                            ChainState *__restrict__ states,
                                                            BlockMap bm,
                                                            int colour, SweepConsts sc, int or_only, Redo rd,
                                                            uint8_t *__restrict__ flags)
{
    half_sweep_body<DIAG, ROWS>(descs, states, bm, colour, sc, or_only, rd, flags);
}

// The same sweep for the unconditional e(T, L) runs (a separate symbol so
// that profiles tell the two workloads apart).
template <int ROWS>
__global__ __launch_bounds__(kBlock) void table_half_sweep_kernel(const ChainDesc *__restrict__ descs,
                                                                  ChainState *__restrict__ states,
                                                                  BlockMap bm, int colour, SweepConsts sc, Redo rd)
{
    half_sweep_body<false, ROWS>(descs, states, bm, colour, sc, 0, rd, nullptr);
}

// The same half-sweep with the gap sites compacted onto consecutive lanes
// (q = 1/2 only).  A block covers CR half-rows x (1024 / CR) sites, two
// site pairs per thread.  Pass 1 (one lane per pair) reads the pairs, draws
// the pair's Philox words and lists the block's gap sites in site order in
// LDS (wave ballots + a prefix over the block's waves); pass 2 runs the
// update for the listed sites, 256 at a time, so sampled sites cost no
// update lanes; pass 3 gives sampled sites of colour 1 their bond energies
// when the sweep's energy is wanted.  Every site gets the arithmetic of the
// plain kernel, so the results are bit-identical to it.
template <bool DIAG, int CR>
__device__ __forceinline__ void half_sweep_compact_body(const ChainDesc *__restrict__ descs,
                                                        ChainState *__restrict__ states,
                                                        BlockMap bm,
                                                        int colour, SweepConsts sc, int or_only, Redo rd,
                                                        uint8_t *__restrict__ flags)
{
    constexpr int PPR = kCompactSites / CR / 2;  // site pairs per block row
    constexpr int NW = kBlock / 64;
    // list entry: Philox words for u and r (top 24 bits each) and the site's
    // index in the block (10 bits: low 8 in the u word, high 2 in the r word)
    __shared__ uint2 gap_list[kCompactSites];
    __shared__ uint16_t fixed_list[kCompactSites];
    __shared__ uint32_t wave_count[2][2][NW];  // [list][pair of the thread][wave]
    __shared__ uint32_t red[2][NW];

    int lb;
    const int c = chain_of_block(bm, (int64_t)blockIdx.x, &lb);
    ChainState *stp = states + c;
    const int phase = stp->phase;
    if (phase == PH_DONE) return;
    const ChainDesc d = descs[c];
    const int nbx = ((d.S >> 1) + PPR - 1) / PPR;
    const int by = lb / nbx;
    const int bx = lb - by * nbx;
    const uint32_t sweep = stp->sweep;
    const float inv_T = stp->inv_T, dscale = stp->dscale;
    const bool want_energy = (colour == 1) && (phase != PH_EQ);
    const bool want_acc = phase != PH_EQ;
    float *const mine_base = colour ? d.h[1] : d.h[0];
    const float *const oth_base = colour ? d.h[0] : d.h[1];
    float *const acc_base = (phase == PH_EQ) ? (colour ? d.acc[1] : d.acc[0]) : nullptr;
    float *const m2_base = acc_base ? (colour ? d.m2[1] : d.m2[0]) : nullptr;

    // pass 1: pairs t and t + 256 of the block; both pairs are read before
    // either draws its random numbers, so that the two loads overlap
    bool gap[2][2], fix[2][2];
    uint32_t wu[2][2], wr[2][2];
    float2 pv[2];
    bool in[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int pi = (int)threadIdx.x + j * kBlock;
        const int y = by * CR + pi / PPR;
        const int h0 = 2 * (bx * PPR + pi % PPR);
        const int s = (y + colour) & 1;
        in[j] = y < d.ny && h0 < ((d.nx - s + 1) >> 1);
        // rows and pairs outside the grid read pair 0 of row 0 instead
        pv[j] = gldi2(mine_base, in[j] ? (uint32_t)(y * d.S + h0) : 0u);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int pi = (int)threadIdx.x + j * kBlock;
        const int y = by * CR + pi / PPR;
        const int h0 = 2 * (bx * PPR + pi % PPR);
        const int s = (y + colour) & 1;
        const bool two = in[j] && (h0 + 1) < ((d.nx - s + 1) >> 1);
        gap[j][0] = in[j] && !is_fixed(pv[j].x);
        gap[j][1] = two && !is_fixed(pv[j].y);
        fix[j][0] = want_energy && in[j] && !gap[j][0];
        fix[j][1] = want_energy && two && !gap[j][1];
        wu[j][0] = wu[j][1] = wr[j][0] = wr[j][1] = 0u;
        if (!or_only && (gap[j][0] || gap[j][1])) {
            const U4 ctr = {(uint32_t)y * (uint32_t)d.nx + (uint32_t)(2 * h0 + s), sweep, d.chain, d.image_id};
            const U4 w = philox4x32_10(ctr, sc.seed_lo, sc.seed_hi);
            wu[j][0] = w.x;
            wr[j][0] = w.y;
            wu[j][1] = w.z;
            wr[j][1] = w.w;
        }
    }
    // positions in the two lists: pair j = 0 of every thread first, then j = 1
    const int lane = (int)(threadIdx.x & 63), wid = (int)(threadIdx.x >> 6);
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    // (the list of sampled sites is only wanted for the sweep's energy: the
    // block-uniform test skips its half of the work in the other half-sweeps)
    uint32_t pre[2][2] = {{0u, 0u}, {0u, 0u}};
#pragma unroll
    for (int L = 0; L < 2; ++L) {
        if (L == 1 && !want_energy) continue;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint64_t b0 = __ballot(L ? fix[j][0] : gap[j][0]);
            const uint64_t b1 = __ballot(L ? fix[j][1] : gap[j][1]);
            pre[L][j] = (uint32_t)(__popcll(b0 & below) + __popcll(b1 & below));
            if (lane == 0) wave_count[L][j][wid] = (uint32_t)(__popcll(b0) + __popcll(b1));
        }
    }
    __syncthreads();
    int n_list[2] = {0, 0};
#pragma unroll
    for (int L = 0; L < 2; ++L) {
        if (L == 1 && !want_energy) continue;
        uint32_t base0 = 0u, base1 = 0u, tot0 = 0u, tot1 = 0u;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const uint32_t c0 = wave_count[L][0][w], c1 = wave_count[L][1][w];
            base0 += (w < wid) ? c0 : 0u;
            base1 += (w < wid) ? c1 : 0u;
            tot0 += c0;
            tot1 += c1;
        }
        n_list[L] = (int)(tot0 + tot1);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            uint32_t pos = (j ? tot0 + base1 : base0) + pre[L][j];
            const uint32_t pi = threadIdx.x + (uint32_t)j * kBlock;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const uint32_t idx = 2u * pi + (uint32_t)k;
                if (L == 0 && gap[j][k]) {
                    gap_list[pos] = make_uint2((wu[j][k] & 0xFFFFFF00u) | (idx & 0xFFu),
                                               (wr[j][k] & 0xFFFFFF00u) | (idx >> 8));
                    ++pos;
                }
                if (L == 1 && fix[j][k]) {
                    fixed_list[pos] = (uint16_t)idx;
                    ++pos;
                }
            }
        }
    }
    __syncthreads();

    // site of a list index: row, half-row position, colour offset, valid neighbours
    auto locate = [&](uint32_t idx, int &y, int &h, int &s, uint32_t &valid) {
        const int pi = (int)(idx >> 1);
        y = by * CR + pi / PPR;
        h = 2 * (bx * PPR + pi % PPR) + (int)(idx & 1u);
        s = (y + colour) & 1;
        const int Wo = (d.nx + s) >> 1;
        valid = (h + s - 1 >= 0 ? 1u : 0u) | (h + s < Wo ? 2u : 0u) | (y > 0 ? 4u : 0u) | (y + 1 < d.ny ? 8u : 0u);
    };
    // all four loads are issued, from clamped positions for missing
    // neighbours (ignored by their valid bits), so that they overlap
    auto neighbours = [&](int y, int h, int s, uint32_t valid, float &nL, float &nR, float &nU, float &nD) {
        const int row = y * d.S;
        nL = angle_of(gldi(oth_base, (uint32_t)(row + max(h + s - 1, 0))));
        nR = angle_of(gldi(oth_base, (uint32_t)(row + min(h + s, d.S - 1))));
        nU = angle_of(gldi(oth_base, (uint32_t)(row + ((valid & 4u) ? -d.S : 0) + h)));
        nD = angle_of(gldi(oth_base, (uint32_t)(row + ((valid & 8u) ? d.S : 0) + h)));
    };

    // a thread sees at most 5 sites (4 gap sites), each below 2^30 in energy units
    uint64_t e_thread = 0u;
    uint32_t acc_thread = 0u;
    // pass 2: the listed gap sites, 256 at a time; the next site's inputs
    // are fetched before the current one is computed (unconditionally, from
    // a clamped list index, so that waiting for the current inputs never
    // waits for these)
    struct Item {
        uint2 e;
        int y, h, s;
        uint32_t valid;
        float a, nL, nR, nU, nD;  // raw words: the sign bit is cleared at use
    };
    auto fetch = [&](int i, Item &it) {
        it.e = gap_list[i];
        locate((it.e.x & 0xFFu) | ((it.e.y & 0xFFu) << 8), it.y, it.h, it.s, it.valid);
        const int row = it.y * d.S;
        it.nL = gldi(oth_base, (uint32_t)(row + max(it.h + it.s - 1, 0)));
        it.nR = gldi(oth_base, (uint32_t)(row + min(it.h + it.s, d.S - 1)));
        it.nU = gldi(oth_base, (uint32_t)(row + ((it.valid & 4u) ? -d.S : 0) + it.h));
        it.nD = gldi(oth_base, (uint32_t)(row + ((it.valid & 8u) ? d.S : 0) + it.h));
        it.a = gldi(mine_base, (uint32_t)(row + it.h));
    };
    const int n_gap = n_list[0];
    Item cur;
    if ((int)threadIdx.x < n_gap) fetch((int)threadIdx.x, cur);
    for (int i = (int)threadIdx.x; i < n_gap; i += kBlock) {
        Item nxt;
        fetch(min(i + kBlock, n_gap - 1), nxt);
        const uint32_t idx = (cur.e.x & 0xFFu) | ((cur.e.y & 0xFFu) << 8);
        const int y = cur.y, h = cur.h, s = cur.s;
        const uint32_t valid = cur.valid;
        const uint32_t site = (uint32_t)(y * d.S + h);
        // the low 8 bits of each word hold the index; unit24 uses the top 24
        const float u = or_only ? 0.5f : unit24(cur.e.x);
        const float r = or_only ? 0.5f : unit24(cur.e.y);
        bool n64 = true;
        const SiteOut o = update_site(angle_of(cur.a), angle_of(cur.nL), angle_of(cur.nR), angle_of(cur.nU),
                                      angle_of(cur.nD), valid, u, r, inv_T, dscale, or_only != 0, &n64);
        cur = nxt;
        if (n64) {  // too close to call: redone in double precision afterwards
            defer_redo(rd, blockIdx.x, kCompactSites / 32, idx);
            continue;
        }
        gsti(mine_base, site, o.phi);
        if (acc_base) accumulate_state_i(acc_base, m2_base, site, o.phi, stp->inv_k, stp->inv_km1);
        acc_thread += o.accepted ? 1u : 0u;
        if (want_energy) e_thread += energy_fx(o.e_bonds);
        if (DIAG && flags) flags[(int64_t)y * d.nx + 2 * h + s] = (uint8_t)o.flags;
    }
    // pass 3: bond energies of the sampled sites of colour 1
    for (int i = (int)threadIdx.x; i < n_list[1]; i += kBlock) {
        int y, h, s;
        uint32_t valid;
        locate((uint32_t)fixed_list[i], y, h, s, valid);
        float nL, nR, nU, nD;
        neighbours(y, h, s, valid, nL, nR, nU, nD);
        const float a = angle_of(gldi(mine_base, (uint32_t)(y * d.S + h)));
        e_thread += energy_fx(bond_energy_half(0.5f * a, nL, nR, nU, nD, valid));
    }
    if (!want_acc) return;
    // wave sums without carries: 64 x 16-bit low parts stay below 2^22, the
    // accepted count (<= 256 per wave) takes bits 22-31, the high parts
    // (< 2^19 per lane) sum in their own word
    uint32_t lo = (uint32_t)(e_thread & 0xFFFFu) | (acc_thread << 22);
    uint32_t hi = (uint32_t)(e_thread >> 16);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo += __shfl_xor(lo, off);
        hi += __shfl_xor(hi, off);
    }
    if (lane == 0) {
        red[0][wid] = lo;
        red[1][wid] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long e = 0ull, a = 0ull;
        for (int i = 0; i < NW; ++i) {
            e += ((unsigned long long)red[1][i] << 16) + (red[0][i] & 0x3FFFFFu);
            a += red[0][i] >> 22;
        }
        if (e) atomicAdd(&stp->e_fx, e);
        if (a) atomicAdd(&stp->acc, a);
    }
}

template <bool DIAG, int CR>
__global__ __launch_bounds__(kBlock) void half_sweep_compact_kernel(const ChainDesc *__restrict__ descs,
                                                                    ChainState *__restrict__ states,
                                                                    BlockMap bm, int colour, SweepConsts sc,
                                                                    int or_only, Redo rd, uint8_t *__restrict__ flags)
{
    half_sweep_compact_body<DIAG, CR>(descs, states, bm, colour, sc, or_only, rd, flags);
}

// The quotients that the control of sweep t needs: 1 + e = (H + N_GP) / N_GP
// with H + N_GP = sum over bonds of (1 - cos), the acceptance ratio and
// (t + 1) / k_a.
struct ControlRatios {
    double ope, A, ta;
};
__device__ __forceinline__ ControlRatios control_ratios(const ChainState &st, const ChainDesc &d, const CtlParams &cp)
{
    return {(double)st.e_fx * cp.e_unit / (double)d.ngp, (double)st.acc / (double)d.P,
            (double)(st.sweep + 1u) / cp.k_a};
}

// Work counters: chain-sweeps, gap-site updates, useful bytes.
__device__ __forceinline__ void count_work(const ChainDesc &d, const CtlParams &cp, unsigned long long *work)
{
    atomicAdd(&work[0], 1ull);
    atomicAdd(&work[1], (unsigned long long)d.P);
    atomicAdd(&work[2], (unsigned long long)(cp.angle_bytes * ((int64_t)d.nx * d.ny + d.P)));
}

// Algorithm 2 steps 5.2-5.5 (relaxation), 6 (equilibrium states) and the
// e(T, L) runs for a chain not done, after both colours of a sweep, on its
// state `st` (in place) with its sums e_fx and acc of that sweep.  The done
// counter (and the work counters) are skipped where null; `slope` gives the
// energy slope at sweep t once the ring buffer holds its energy.  (1 / T stays
// as the host set it.)
template <class Slope>
__device__ __forceinline__ void control_core(ChainState &st, const ChainDesc &d, const CtlParams &cp,
                                             const ControlRatios &r, unsigned int *done_count,
                                             unsigned long long *work, Slope slope)
{
    if (work) count_work(d, cp, work);
    const uint32_t t = st.sweep;
    st.acc = 0ull;
    st.e_fx = 0ull;
    if (st.phase == PH_RELAX) {
        if (r.A < cp.a_targ) st.a_relax = 1.0 + r.ta;
        st.ring[t % (uint32_t)cp.n_fit] = r.ope;
        if (t >= (uint32_t)cp.n_fit && t % (uint32_t)cp.n_f == 0u) st.k = slope(t);
        st.A_last = r.A;
        const uint32_t tn = t + 1u;
        st.sweep = tn;
        bool stop;
        if (cp.fixed_relax >= 0) stop = tn >= (uint32_t)cp.fixed_relax;
        else stop = !(st.k < 0.0 && (int64_t)tn <= (int64_t)cp.i_max);
        st.a_cur = st.a_relax;
        if (stop) {
            st.relax_sweeps = (int32_t)tn;
            st.not_converged = (cp.fixed_relax < 0 && st.k < 0.0) ? 1 : 0;
            st.eq_left = cp.K;
            st.phase = cp.K > 0 ? PH_EQ : PH_DONE;
            st.a_cur = cp.eq_a_mode ? st.a_relax : 1.0;
            st.inv_k = 1.0f;
            st.inv_km1 = 0.0f;
            st.inv_k_d = 1.0;
            st.inv_km1_d = 0.0;
        }
    } else if (st.phase == PH_EQ) {
        st.sweep = t + 1u;
        if (--st.eq_left <= 0) {
            st.phase = PH_DONE;
        } else {
            const int k = cp.K - st.eq_left + 1;  // the next sweep's state number
            st.inv_k = 1.0f / (float)k;
            st.inv_km1 = 1.0f / (float)(k - 1);
            st.inv_k_d = 1.0 / (double)k;
            st.inv_km1_d = 1.0 / (double)(k - 1);
        }
    } else {  // PH_TABLE
        if (r.A < cp.a_targ) st.a_relax = 1.0 + r.ta;
        st.a_cur = st.a_relax;
        if ((int64_t)t >= (int64_t)cp.burn) st.e_sum += r.ope;
        st.sweep = t + 1u;
        if ((int64_t)t + 1 >= (int64_t)cp.burn + cp.meas) st.phase = PH_DONE;
    }
    st.dscale = (float)(kTwoPi * cp.q / st.a_cur);
    if (st.phase == PH_DONE && done_count) atomicAdd(done_count, 1u);
}

// The control of chain c of a chain set (control_core on its state in place:
// a copy would put the ring buffer in scratch memory).
__device__ __forceinline__ void control_chain(const ChainDesc *__restrict__ descs, ChainState *__restrict__ states,
                                              int c, const CtlParams &cp, unsigned int *done_count,
                                              unsigned long long *work)
{
    ChainState &st = states[c];
    if (st.phase == PH_DONE) return;
    const ChainDesc d = descs[c];
    control_core(st, d, cp, control_ratios(st, d, cp), done_count, work, [&](uint32_t t) { return ring_slope(st.ring, t, cp.n_fit, cp.w); });
}

// The deferred double-precision updates of one half-sweep (block shape
// `rows`, `compact`): each flagged site is redone by update_site_d from the
// inputs the sweep saw (it left the site unchanged), with the same random
// numbers, written back in single precision, and its accepted count and
// bond energy added to its chain.  A wave takes one bitmap word (32 sweep
// blocks) at a time; its lanes split over (flagged block, mask word), 64 /
// words blocks per pass, and a lane redoes the sites of its mask word.  The
// bits are cleared on the way, so the buffers are zero again for the next
// half-sweep.  With `ctl` set (after the colour-1 half-sweep) the last block
// to finish also runs the per-sweep control of all n_all chains, which saves
// the control kernel's launch; it finds out that it is last from the ticket
// counter, which it resets.
struct FusedControl {
    CtlParams cp;
    unsigned int *ticket;  // zero before the first launch; the last block resets it
    unsigned int *done_count;
    unsigned long long *work;
    int32_t n_all;
    int32_t on;
};

template <bool DIAG>
__global__ __launch_bounds__(kBlock) void redo_fp64_kernel(const ChainDesc *__restrict__ descs,
                                                           ChainState *__restrict__ states,
                                                           BlockMap bm,
                                                           int64_t total_blocks, int rows, int compact, int colour,
                                                           SweepConsts sc, int or_only, Redo rd,
                                                           uint8_t *__restrict__ flags, FusedControl ctl)
{
    const int words = compact ? kCompactSites / 32 : 2 * kBlock / 32;  // 32 or 16
    const int per = 64 / words;                                         // blocks per pass
    const int ppr = compact ? kCompactSites / rows / 2 : kBlock / rows;  // site pairs per block row
    const int64_t nw = (total_blocks + 31) >> 5;
    const int lane = (int)(threadIdx.x & 63);
    const int slot = lane / words, k = lane % words;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t wi = wave; wi < nw; wi += n_waves) {
        uint32_t bits = rd.blocks[wi];
        if (!bits) continue;
        if (lane == 0) rd.blocks[wi] = 0u;
        while (bits) {
            // this lane's block: the slot-th lowest set bit of this pass
            uint32_t b = bits;
            for (int i = 0; i < slot; ++i) b &= b - 1u;
            for (int i = 0; i < per; ++i) bits &= bits - 1u;
            if (!b) continue;
            const int64_t gb = (wi << 5) + (__ffs(b) - 1);
            uint32_t m = rd.mask[gb * words + k];
            if (!m) continue;
            rd.mask[gb * words + k] = 0u;
            int lb;
            const int c = chain_of_block(bm, gb, &lb);
            ChainState *stp = states + c;
            const ChainDesc d = descs[c];
            const int nbx = ((d.S >> 1) + ppr - 1) / ppr;
            const int by = lb / nbx;
            const int bx = lb - by * nbx;
            const int phase = stp->phase;
            const bool want_energy = (colour == 1) && (phase != PH_EQ);
            const bool want_acc = phase != PH_EQ;
            float *mine = colour ? d.h[1] : d.h[0];
            const float *oth = colour ? d.h[0] : d.h[1];
            float *accp = (phase == PH_EQ) ? (colour ? d.acc[1] : d.acc[0]) : nullptr;
            float *m2p = accp ? (colour ? d.m2[1] : d.m2[0]) : nullptr;
            while (m) {
                const int bit = __ffs(m) - 1;
                m &= m - 1u;
                const int idx = 32 * k + bit;
                const int pi = idx >> 1, sl = idx & 1;
                const int y = by * rows + pi / ppr;
                const int h = 2 * (bx * ppr + pi % ppr) + sl;
                const int s = (y + colour) & 1;
                const int Wo = (d.nx + s) >> 1;
                const uint32_t valid = (h + s - 1 >= 0 ? 1u : 0u) | (h + s < Wo ? 2u : 0u) |
                                       (y > 0 ? 4u : 0u) | (y + 1 < d.ny ? 8u : 0u);
                const float *orow = oth + (int64_t)y * d.S;
                const float nL = (valid & 1u) ? angle_of(orow[h + s - 1]) : 0.0f;
                const float nR = (valid & 2u) ? angle_of(orow[h + s]) : 0.0f;
                const float nU = (valid & 4u) ? angle_of(orow[h - d.S]) : 0.0f;
                const float nD = (valid & 8u) ? angle_of(orow[h + d.S]) : 0.0f;
                float *mp = mine + (int64_t)y * d.S + h;
                const float a = angle_of(*mp);
                float u = 0.5f, r = 0.5f;
                if (!or_only) {
                    const U4 ctr = {(uint32_t)y * (uint32_t)d.nx + (uint32_t)(2 * (h & ~1) + s), stp->sweep,
                                    d.chain, d.image_id};
                    const U4 wd = philox4x32_10(ctr, sc.seed_lo, sc.seed_hi);
                    u = unit24(sl ? wd.z : wd.x);
                    r = unit24(sl ? wd.w : wd.y);
                }
                const SiteOutD o = update_site_d((double)a, (double)nL, (double)nR, (double)nU, (double)nD, valid,
                                                 (double)u, (double)r, stp->a_cur, stp->T, sc.q64,
                                                 or_only != 0);
                const float out = (float)o.phi;
                *mp = out;
                if (accp)
                    accumulate_state(accp + (int64_t)y * d.S + h, m2p ? m2p + (int64_t)y * d.S + h : nullptr, out,
                                     stp->inv_k, stp->inv_km1);
                if (want_acc && o.accepted) atomicAdd(&stp->acc, 1ull);
                if (want_energy) atomicAdd(&stp->e_fx, (unsigned long long)energy_fx((float)o.e_bonds));
                if (DIAG && flags) flags[(int64_t)y * d.nx + 2 * h + s] = (uint8_t)o.flags;
            }
        }
    }
    if (!ctl.on) return;
    __shared__ int last;
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        last = atomicAdd(ctl.ticket, 1u) == gridDim.x - 1u;
    }
    __syncthreads();
    if (!last) return;
    __threadfence();  // the other blocks' counts and energies are visible
    for (int c = (int)threadIdx.x; c < ctl.n_all; c += (int)blockDim.x)
        control_chain(descs, states, c, ctl.cp, ctl.done_count, ctl.work);
    if (threadIdx.x == 0) *ctl.ticket = 0u;
}

// Relaxed device-scope loads (coherent between the XCDs).
__device__ __forceinline__ uint32_t ld_agent(const unsigned int *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned long long ld_agent64(const unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum over a wave in lane 63, by row shifts and row broadcasts on the vector
// unit (a butterfly through LDS takes 6 round trips of some 100 cycles).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_get(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ void dpp_step(unsigned long long &e, uint32_t &a)
{
    const uint32_t lo = dpp_get<CTRL, ROWS>((uint32_t)e), hi = dpp_get<CTRL, ROWS>((uint32_t)(e >> 32));
    e += ((unsigned long long)hi << 32) | lo;
    a += dpp_get<CTRL, ROWS>(a);
}
__device__ __forceinline__ void wave_sum_63(unsigned long long &e, uint32_t &a)
{
    dpp_step<0x111, 0xF>(e, a);  // row_shr:1
    dpp_step<0x112, 0xF>(e, a);  // row_shr:2
    dpp_step<0x114, 0xF>(e, a);  // row_shr:4
    dpp_step<0x118, 0xF>(e, a);  // row_shr:8
    dpp_step<0x142, 0xA>(e, a);  // row_bcast:15 into rows 1 and 3
    dpp_step<0x143, 0xC>(e, a);  // row_bcast:31 into rows 2 and 3
}
__device__ __forceinline__ unsigned long long readlane64(unsigned long long v, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return ((unsigned long long)hi << 32) | lo;
}

// ring_slope by a whole wave: lane j loads the j-th value (the newest is
// `newest`, not yet in the ring), the sum runs in the same order.
__device__ __forceinline__ double ring_slope_wave(const double *ring, double newest, uint32_t t, int n_fit,
                                                  const double *w, int lane)
{
    const int j0 = lane < n_fit ? lane : 0;
    const double r = j0 == n_fit - 1 ? newest : ring[(t + 1u + (uint32_t)j0) % (uint32_t)n_fit];
    const double wl = w[j0];
    const int rl = __double2loint(r), rh = __double2hiint(r), wlo = __double2loint(wl), whi = __double2hiint(wl);
    double s = 0.0;
    for (int j = 0; j < n_fit; ++j) {
        const double rj = __hiloint2double(__builtin_amdgcn_readlane(rh, j), __builtin_amdgcn_readlane(rl, j));
        const double wj = __hiloint2double(__builtin_amdgcn_readlane(whi, j), __builtin_amdgcn_readlane(wlo, j));
        s += wj * rj;
    }
    return s;
}

// ================================================================ fused tile sweep
// A whole sweep in one launch.  A block stages one tile of both colours in
// LDS: TH rows x 2 kTileH columns of the grid (kTileH half-columns per
// colour) plus a halo of two rows and columns.  It updates colour 0 on the
// tile and on the ring of sites around it, then colour 1 on the tile, which
// so sees the colour-0 values of its neighbours after their update (the ring
// repeats updates that the neighbouring tiles also make, with the same
// inputs and the same random numbers, so with the same results).  Decisions
// too close to call in single precision are redone in double precision in
// the block after each colour, before anything reads them.  The gap sites
// of the tile are then written to the chain's second half-grids (h2):
// reading h and writing h2 keeps every tile's halo at the state before the
// sweep while other tiles store theirs.  control_kernel then swaps h and h2
// of every chain swept (one thread per chain: no block of the sweep waits
// for the others) before it runs the per-sweep control; a launch of at most
// a few thousand blocks does both in its last block instead.
//
// Within a colour the gap sites are listed in LDS first (wave ballots; each
// wave lists the candidates it read, interleaved with the other waves at 64
// sites, and updates its own list), so that lanes only do gap sites; with
// the sweep's energy wanted, the colour-1 sampled sites of the tile get a
// second list for their bond energies.  Every site gets update_site, the
// arithmetic of the half-sweep kernels, so the results equal theirs bit for
// bit.  `mode` 0 is the full sweep; 1 and 2 update only colour 0 or 1, in
// place (no tile reads a value another tile writes then), for the
// single-colour diagnostics.
constexpr int kTileH = 64;                // half-columns per tile and colour
constexpr int kTileLS = kTileH + 8;       // LDS row: half-columns hx0 - 4 .. hx0 + kTileH + 3
constexpr int kTileNW = kBlock / 64;      // waves per block
// Fused sweeps of at most this many blocks run the control themselves (a
// chain's last block, found by a returning atomic that every block waits for
// at its end).  A batch of 24 images of 128 to 1024 a side: 24.4 ms a fill with
// control_kernel after every sweep, 20.2 ms without; at 44032 blocks (sixteen
// chains of 4096^2) 250.1 and 250.6 ms, and the atomics only grow from there.
constexpr int64_t kTileCtlMaxBlocks = 16384;

// The double-precision decision of one tile site (colour c, local row r,
// half-column j) from its LDS inputs: the steps of redo_fp64_kernel.  Kept
// out of line, so that the sweep's loops do not hold the double update's
// constants in registers.
__device__ __noinline__ SiteOutD tile_redo_site(const float *a, int rows, int c, int r, int j, int y0, int hx0, int nx,
                                                int ny, uint32_t sweep, uint32_t chain, uint32_t image_id,
                                                SweepConsts sc, int or_only, double a_cur, double T)
{
    const float *own = a + ((size_t)c * rows + r) * kTileLS + j;
    const float *oth = a + ((size_t)(c ^ 1) * rows + r) * kTileLS + j;
    const int s = (r + c) & 1;
    const int y = y0 - 2 + r, h = hx0 - 4 + j;
    const int Wo = (nx + s) >> 1;
    const uint32_t valid = (h + s - 1 >= 0 ? 1u : 0u) | (h + s < Wo ? 2u : 0u) | (y > 0 ? 4u : 0u) |
                           (y + 1 < ny ? 8u : 0u);
    const float nL = (valid & 1u) ? angle_of(oth[s - 1]) : 0.0f;
    const float nR = (valid & 2u) ? angle_of(oth[s]) : 0.0f;
    const float nU = (valid & 4u) ? angle_of(oth[-kTileLS]) : 0.0f;
    const float nD = (valid & 8u) ? angle_of(oth[kTileLS]) : 0.0f;
    float u = 0.5f, rr = 0.5f;
    if (!or_only) {
        const U4 ctr = {(uint32_t)y * (uint32_t)nx + (uint32_t)(2 * (h & ~1) + s), sweep, chain, image_id};
        const U4 w = philox4x32_10(ctr, sc.seed_lo, sc.seed_hi);
        const bool second = (h & 1) != 0;
        u = unit24(second ? w.z : w.x);
        rr = unit24(second ? w.w : w.y);
    }
    return update_site_d((double)angle_of(*own), (double)nL, (double)nR, (double)nU, (double)nD, valid, (double)u,
                         (double)rr, a_cur, T, sc.q64, or_only != 0);
}

// The parameters one sweep of a chain reads (written by the control between
// sweeps).
struct SweepState {
    int32_t phase;
    uint32_t sweep;
    float inv_T, dscale, inv_k, inv_km1;
    double T, a_cur;
};

__device__ __forceinline__ SweepState sweep_state_of(const ChainState *stp)
{
    SweepState s;
    s.phase = stp->phase;
    s.sweep = stp->sweep;
    s.inv_T = stp->inv_T;
    s.dscale = stp->dscale;
    s.inv_k = stp->inv_k;
    s.inv_km1 = stp->inv_km1;
    s.T = stp->T;
    s.a_cur = stp->a_cur;
    return s;
}

template <int TH>
struct TileShared {
    static constexpr int NW = kTileNW;
    // list entries per wave: its rows of the colour-0 pass with the ring
    // (TH + 2 rows of kTileH columns, a row per wave in turn) and its share
    // of the ring's two side columns (at most 64 per wave)
    static constexpr int CAP = (TH + 2 + NW - 1) / NW * 64 + 64;
    static constexpr int RW = ((TH + 4) * kTileLS + 31) / 32;     // redo bitmap words
    alignas(16) float a[2][TH + 4][kTileLS];  // angle words (sign bit: sampled), colour, row, half-column
    // per wave: gap entries from the front, sampled entries from the back;
    // entry = local row << 7 | local half-column
    uint16_t list[NW][CAP];
    uint32_t redo[RW];
    uint32_t red[3][NW];
    int any_redo[2];
};

// Stages the tile and its halo (both colours, 18 float4 per row and colour;
// the colour loop outside, so that the base pointer of every load is
// uniform) from h into LDS.  No barrier at the end.
template <int TH>
__device__ __forceinline__ void tile_stage(TileShared<TH> &L, const ChainDesc &d, int y0, int hx0)
{
    constexpr int NT = kBlock;
    const int tid = (int)threadIdx.x;
    constexpr int NQ = kTileLS / 4;
    constexpr int NLOAD = (TH + 4) * NQ;
    constexpr int IT = (NLOAD + NT - 1) / NT;
    v4f v[2][IT];
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
        const float *src = cc ? d.h[1] : d.h[0];
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int k = tid + it * NT;
            const int r = k / NQ, q = k - r * NQ;
            const int y = y0 - 2 + r, h = hx0 - 4 + 4 * q;
            const bool in = k < NLOAD && y >= 0 && y < d.ny && h >= 0 && h < d.S;
            // outside the grid: zeros, never a candidate (EDGE bounds)
            // nor a valid neighbour
            v[cc][it] = gldi4(src, in ? (uint32_t)(y * d.S + h) : 0u);
            if (!in) v[cc][it] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        }
    }
#pragma unroll
    for (int cc = 0; cc < 2; ++cc)
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int k = tid + it * NT;
            const int r = k / NQ, q = k - r * NQ;
            if (k < NLOAD) *(v4f *)&L.a[cc][r][4 * q] = v[cc][it];
        }
}

// The sweep (mode 0) or one colour (modes 1, 2) of a staged tile, and the
// write-back of its gap sites and equilibrium sums.
template <bool DIAG, int TH, bool EDGE>
__device__ __forceinline__ void tile_update(TileShared<TH> &L, const ChainDesc &d, const SweepState &ss, int y0, int hx0,
                                            int mode, const SweepConsts &sc, int or_only, uint8_t *__restrict__ flags,
                                            uint64_t &e_thread, uint32_t &acc_thread)
{
    constexpr int NT = kBlock, NW = kTileNW;
    // the wave index through readfirstlane: the compiler then knows it is
    // uniform, and keeps the row loops of the list building and their
    // counters on the scalar unit
    const int tid = (int)threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int phase = ss.phase;
    const uint32_t sweep = ss.sweep;
    const float inv_T = ss.inv_T, dscale = ss.dscale;
    const bool eq = phase == PH_EQ;
    float *const dst0 = mode == 0 ? d.h2[0] : d.h[0];
    float *const dst1 = mode == 0 ? d.h2[1] : d.h[1];

    // the tile's gap sites of colour cc to the destination half-grid
    // (16-byte groups holding at least one gap site), and the equilibrium sums
    auto write_back = [&](int cc) {
        constexpr int NQ = kTileH / 4;
        const float ik = ss.inv_k, ikm1 = ss.inv_km1;
        float *const dst = cc ? dst1 : dst0;
        float *const ap = eq ? (cc ? d.acc[1] : d.acc[0]) : nullptr;
        float *const mp = cc ? d.m2[1] : d.m2[0];
        for (int k = tid; k < TH * NQ; k += NT) {
            const int rr = k / NQ, q = k - rr * NQ;
            const int y = y0 + rr;
            if (y >= d.ny) continue;
            const int h = hx0 + 4 * q;
            const v4f v = *(const v4f *)&L.a[cc][rr + 2][4 + 4 * q];
            const bool g0 = !is_fixed(v.x), g1 = !is_fixed(v.y), g2 = !is_fixed(v.z), g3 = !is_fixed(v.w);
            if (!(g0 || g1 || g2 || g3)) continue;
            const uint32_t idx = (uint32_t)(y * d.S + h);
            gsti4(dst, idx, v);
            if (ap) {
                // the group's gap sites into the equilibrium sums (and the
                // squared deviations), the arithmetic of accumulate_state,
                // with 16-byte loads and stores; the other elements keep
                // their values
                const int W = (d.nx - ((y + cc) & 1) + 1) >> 1;
                const bool gg[4] = {g0, g1, g2, g3};
                const v4f s0 = gldi4(ap, idx);
                v4f s1 = s0;
                v4f m = mp ? gldi4(mp, idx) : v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (gg[e] && h + e < W) {
                        s1[e] = s0[e] + v[e];
                        m[e] = fmaf(v[e] - s0[e] * ikm1, v[e] - s1[e] * ik, m[e]);
                    }
                gsti4(ap, idx, s1);
                if (mp) gsti4(mp, idx, m);
            }
        }
    };

    const int npass = mode == 0 ? 2 : 1;
    for (int pass = 0; pass < npass; ++pass) {
        const int c = mode == 0 ? pass : mode - 1;
        const bool ring = mode == 0 && c == 0;       // colour 0 of a full sweep: tile and ring
        const bool energy = c == 1 && !eq;           // the sweep's energy comes from colour 1
        const int r_lo = ring ? 1 : 2, r_hi = TH + (ring ? 3 : 2);
        uint16_t *lst = L.list[wid];
        // List the gap sites (and, for the energy, the sampled sites): a
        // wave takes one row at a time, lane l its tile column j = 4 + l;
        // with the ring, the last wave (which has the fewest rows) then takes
        // the ring's sites beside the tile, of which colour 1 reads one per
        // row (16 chains of 4096^2, 66% missing: 228.6 ms a fill, 232.7 with
        // both sides of every row, dealt to the first waves).  A site in the tile is either a gap or a
        // sample, so a lane's rank among the sampled lanes is its rank among
        // the lanes holding a site less its rank among the gap lanes: one
        // ballot per row.  FULL: every lane of the wave holds a site (the
        // interior rows of an interior tile), so that rank among them is the
        // lane index.
        int ng = 0, ns = 0;
        auto add = [&](auto FULL, bool cand, int r, int j) {
            constexpr bool full = decltype(FULL)::value;
            bool in = cand, gap = false;
            if (cand) {
                const float v = L.a[c][r][j];
                if (EDGE) {
                    const int y = y0 - 2 + r, h = hx0 - 4 + j, s = (r + c) & 1;
                    in = y < d.ny && y >= 0 && h >= 0 && h < ((d.nx - s + 1) >> 1);
                }
                gap = in && !is_fixed(v);
            }
            const uint16_t ent = (uint16_t)((r << 7) | j);
            const uint64_t bg = __ballot(gap);
            const int rg = rank_below(bg);
            if (gap) lst[ng + rg] = ent;
            const int cg = __popcll(bg);
            ng += cg;
            if (energy) {
                const uint64_t bi = full ? ~0ull : __ballot(in);
                const int rs = (full ? lane : rank_below(bi)) - rg;
                if (in && !gap) lst[TileShared<TH>::CAP - 1 - (ns + rs)] = ent;
                ns += (full ? 64 : __popcll(bi)) - cg;
            }
        };
        for (int r = r_lo + wid; r < r_hi; r += NW) add(std::integral_constant<bool, !EDGE>{}, true, r, 4 + lane);
        if (ring && wid == NW - 1) {
            const int r = 2 + (lane < TH ? lane : 0);
            add(std::false_type{}, lane < TH, r, (r & 1) ? 3 : kTileH + 4);
        }
        __syncthreads();
        // the listed gap sites
        for (int e = lane; e < ng; e += 64) {
            const uint32_t ent = lst[e];
            const int r = (int)(ent >> 7), j = (int)(ent & 127u);
            const int s = (r + c) & 1;  // y0 is even
            const float *oth = &L.a[c ^ 1][r][j];
            const float a0 = L.a[c][r][j];
            const float nL = angle_of(oth[s - 1]), nR = angle_of(oth[s]);
            const float nU = angle_of(oth[-kTileLS]), nD = angle_of(oth[kTileLS]);
            const int y = y0 - 2 + r, h = hx0 - 4 + j;
            uint32_t valid = 15u;
            if (EDGE) {
                const int Wo = (d.nx + s) >> 1;
                valid = (h + s - 1 >= 0 ? 1u : 0u) | (h + s < Wo ? 2u : 0u) | (y > 0 ? 4u : 0u) |
                        (y + 1 < d.ny ? 8u : 0u);
            }
            float u = 0.5f, rr = 0.5f;
            if (!or_only) {
                const U4 ctr = {(uint32_t)y * (uint32_t)d.nx + (uint32_t)(2 * (h & ~1) + s), sweep, d.chain,
                                d.image_id};
                const U4 w = philox4x32_10(ctr, sc.seed_lo, sc.seed_hi);
                const bool second = (h & 1) != 0;
                u = unit24(second ? w.z : w.x);
                rr = unit24(second ? w.w : w.y);
            }
            bool n64 = true;
            const SiteOut o = update_site(a0, nL, nR, nU, nD, valid, u, rr, inv_T, dscale, or_only != 0, &n64);
            if (n64) {  // too close to call: redone in double precision below
                const int wi = r * kTileLS + j;
                atomicOr(&L.redo[wi >> 5], 1u << (wi & 31));
                L.any_redo[pass] = 1;
                continue;
            }
            L.a[c][r][j] = o.phi;
            const bool own = !ring || (r >= 2 && r < TH + 2 && j >= 4 && j < kTileH + 4);
            if (own) {
                acc_thread += o.accepted ? 1u : 0u;
                if (energy) e_thread += energy_fx(o.e_bonds);
                if (DIAG && flags) flags[(int64_t)y * d.nx + 2 * h + s] = (uint8_t)o.flags;
            }
        }
        // bond energies of the tile's sampled colour-1 sites
        for (int e = lane; e < ns; e += 64) {
            const uint32_t ent = lst[TileShared<TH>::CAP - 1 - e];
            const int r = (int)(ent >> 7), j = (int)(ent & 127u);
            const int s = (r + c) & 1;
            const float *oth = &L.a[c ^ 1][r][j];
            const float nL = angle_of(oth[s - 1]), nR = angle_of(oth[s]);
            const float nU = angle_of(oth[-kTileLS]), nD = angle_of(oth[kTileLS]);
            uint32_t valid = 15u;
            if (EDGE) {
                const int y = y0 - 2 + r, h = hx0 - 4 + j;
                const int Wo = (d.nx + s) >> 1;
                valid = (h + s - 1 >= 0 ? 1u : 0u) | (h + s < Wo ? 2u : 0u) | (y > 0 ? 4u : 0u) |
                        (y + 1 < d.ny ? 8u : 0u);
            }
            e_thread += energy_fx(bond_energy_half(0.5f * angle_of(L.a[c][r][j]), nL, nR, nU, nD, valid));
        }
        __syncthreads();
        // the deferred decisions, in double precision from the same inputs
        if (L.any_redo[pass]) {
            for (int wd = tid; wd < TileShared<TH>::RW; wd += NT) {
                uint32_t m = L.redo[wd];
                if (!m) continue;
                L.redo[wd] = 0u;
                while (m) {
                    const int wi = wd * 32 + __ffs(m) - 1;
                    m &= m - 1u;
                    const int r = wi / kTileLS, j = wi - r * kTileLS;
                    const SiteOutD o = tile_redo_site(&L.a[0][0][0], TH + 4, c, r, j, y0, hx0, d.nx, d.ny, sweep, d.chain,
                                                      d.image_id, sc, or_only, ss.a_cur, ss.T);
                    const int y = y0 - 2 + r, h = hx0 - 4 + j, s = (r + c) & 1;
                    L.a[c][r][j] = (float)o.phi;
                    const bool own = !ring || (r >= 2 && r < TH + 2 && j >= 4 && j < kTileH + 4);
                    if (own) {
                        acc_thread += o.accepted ? 1u : 0u;
                        if (energy) e_thread += energy_fx((float)o.e_bonds);
                        if (DIAG && flags) flags[(int64_t)y * d.nx + 2 * h + s] = (uint8_t)o.flags;
                    }
                }
            }
            __syncthreads();
        }
        if (mode == 0 && pass == 0) write_back(0);
    }

    // the colour not written back after its own pass (colour 0 of a full
    // sweep is final once its pass is done: colour 1 only reads it)
    write_back(mode == 1 ? 0 : 1);
}

// Stage, then sweep, the tile of a one-launch-per-sweep kernel.
template <bool DIAG, int TH, bool EDGE>
__device__ __forceinline__ void tile_sweep_body(TileShared<TH> &L, const ChainDesc &d, const SweepState &ss, int y0,
                                                int hx0, int mode, const SweepConsts &sc, int or_only,
                                                uint8_t *__restrict__ flags, uint64_t &e_thread,
                                                uint32_t &acc_thread)
{
    tile_stage(L, d, y0, hx0);
    __syncthreads();
    tile_update<DIAG, TH, EDGE>(L, d, ss, y0, hx0, mode, sc, or_only, flags, e_thread, acc_thread);
}

// The block's bond energy and accepted count added to its chain (energy in
// 16-bit halves, so that the 32-bit lane sums cannot carry out).  With
// `arrive` the accepted counter also counts the chain's blocks in its upper
// bits, and the value it had before this block is returned to wave 0.  Called
// by every thread of the block.
constexpr int kArriveShift = 40;  // a chain has at most 2^31 sites
template <int TH>
__device__ __forceinline__ unsigned long long tile_block_sums(TileShared<TH> &L, uint64_t e_thread, uint32_t acc_thread,
                                                              unsigned long long *e_sum, unsigned long long *acc_sum,
                                                              bool wanted, bool arrive)
{
    const int tid = (int)threadIdx.x;
    constexpr int NW = kTileNW;
    const int wid = tid >> 6;
    if (wanted) {
        uint32_t lo = (uint32_t)(e_thread & 0xFFFFu), hi = (uint32_t)(e_thread >> 16), ac = acc_thread;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            lo += __shfl_xor(lo, off);
            hi += __shfl_xor(hi, off);
            ac += __shfl_xor(ac, off);
        }
        if ((tid & 63) == 0) {
            L.red[0][wid] = lo;
            L.red[1][wid] = hi;
            L.red[2][wid] = ac;
        }
    }
    __syncthreads();
    unsigned long long before = 0ull;
    if (tid == 0) {
        unsigned long long e = 0ull, a = 0ull;
        if (wanted)
            for (int i = 0; i < NW; ++i) {
                e += ((unsigned long long)L.red[1][i] << 16) + L.red[0][i];
                a += L.red[2][i];
            }
        if (arrive) {
            // the energy is added before the block counts as arrived: the
            // first addition's result is waited for
            if (e) {
                const unsigned long long old = atomicAdd(e_sum, e);
                __asm__ volatile("" ::"v"((uint32_t)old), "v"((uint32_t)(old >> 32)) : "memory");
            }
            before = atomicAdd(acc_sum, a | (1ull << kArriveShift)) + a;
        } else {
            if (e) atomicAdd(e_sum, e);
            if (a) atomicAdd(acc_sum, a);
        }
    }
    return before;
}

// The end of a chain's sweep, by wave 0 of its last block: h and h2 exchanged
// (the chain's `swapped` flag toggled) and the per-sweep control, from the
// chain's energy and accepted count.  Only the next launch reads h2, so no
// fence is needed.
__device__ __forceinline__ void chain_end(ChainDesc &dd, ChainState &st, const ChainDesc &d, unsigned long long acc,
                                          const FusedControl &ctl)
{
    const int lane = (int)(threadIdx.x & 63);
    const unsigned long long e = ld_agent64(&st.e_fx);
    const uint32_t t = st.sweep;
    // the control's three quotients by one division, a lane each
    const double num = lane == 0 ? (double)e * ctl.cp.e_unit : lane == 1 ? (double)acc : (double)(t + 1u);
    const double den = lane == 0 ? (double)d.ngp : lane == 1 ? (double)d.P : ctl.cp.k_a;
    const unsigned long long quo = (unsigned long long)__double_as_longlong(num / den);
    ControlRatios r;
    r.ope = __longlong_as_double((long long)readlane64(quo, 0));
    r.A = __longlong_as_double((long long)readlane64(quo, 1));
    r.ta = __longlong_as_double((long long)readlane64(quo, 2));
    double slope = 0.0;
    if (st.phase == PH_RELAX && t >= (uint32_t)ctl.cp.n_fit && t % (uint32_t)ctl.cp.n_f == 0u)
        slope = ring_slope_wave(st.ring, r.ope, t, ctl.cp.n_fit, ctl.cp.w, lane);
    if (lane == 0) {
        dd.h[0] = d.h2[0];
        dd.h[1] = d.h2[1];
        dd.h2[0] = d.h[0];
        dd.h2[1] = d.h[1];
        st.swapped ^= 1;
        control_core(st, d, ctl.cp, r, ctl.done_count, ctl.work, [&](uint32_t) { return slope; });
    }
}

// With `ctl.on` a chain's last block to finish also ends its sweep
// (chain_end), which saves the control kernel: the blocks of a chain count
// themselves in the upper bits of its accepted counter, so that no counter is
// shared between chains.
template <bool DIAG, int TH>
__global__ __launch_bounds__(kBlock) void sweep_tile_kernel(ChainDesc *__restrict__ descs,
                                                            ChainState *__restrict__ states, BlockMap bm,
                                                            int mode, SweepConsts sc, int or_only,
                                                            uint8_t *__restrict__ flags, FusedControl ctl)
{
    __shared__ TileShared<TH> L;
    const int tid = (int)threadIdx.x;
    for (int w = tid; w < TileShared<TH>::RW; w += kBlock) L.redo[w] = 0u;
    if (tid < 2) L.any_redo[tid] = 0;
    // blocks go round-robin to the 8 XCDs: give each XCD a contiguous run of
    // tiles, so that the halo rows tiles share are read through one L2
    const uint32_t G = gridDim.x, b = blockIdx.x;
    const uint32_t per = G >> 3, rem = G & 7u, xcd = b & 7u;
    const int64_t lbk = (int64_t)xcd * per + (int64_t)min(xcd, rem) + (int64_t)(b >> 3);
    int lb;
    const int cid = chain_of_block(bm, lbk, &lb);
    ChainState *stp = states + cid;
    uint64_t e_thread = 0u;
    uint32_t acc_thread = 0u;
    const int phase = stp->phase;
    if (phase != PH_DONE) {
        const ChainDesc d = descs[cid];
        const int nbx = d.S / kTileH;
        const int ty = lb / nbx, tx = lb - ty * nbx;
        const int y0 = ty * TH, hx0 = tx * kTileH;
        const bool edge = !(ty >= 1 && y0 + TH + 2 <= d.ny && tx >= 1 && hx0 + kTileH + 2 <= (d.nx >> 1));
        __syncthreads();
        const SweepState ss = sweep_state_of(stp);
        if (edge)
            tile_sweep_body<DIAG, TH, true>(L, d, ss, y0, hx0, mode, sc, or_only, flags, e_thread, acc_thread);
        else
            tile_sweep_body<DIAG, TH, false>(L, d, ss, y0, hx0, mode, sc, or_only, flags, e_thread, acc_thread);
        const bool arrive = ctl.on != 0;
        if (arrive || phase != PH_EQ) {
            unsigned long long before = tile_block_sums(L, e_thread, acc_thread, &stp->e_fx, &stp->acc,
                                                        phase != PH_EQ, arrive);
            if (arrive && tid < 64) {
                before = readlane64(before, 0);
                const unsigned long long blocks = (unsigned long long)nbx * (unsigned long long)((d.ny + TH - 1) / TH);
                if ((before >> kArriveShift) == blocks - 1ull)
                    chain_end(descs[cid], states[cid], d, before & ((1ull << kArriveShift) - 1ull), ctl);
            }
        }
    }
}

// Many fused sweeps per cooperative launch, for chain sets whose tiles the GPU
// holds at once: a 1024 x 1024 chain is 256 tiles of 32 rows.  A block keeps its tile (TH rows
// x 2 kTileH columns, both colours) in LDS from the launch's first sweep to
// its last, and exchanges only the sites around it with the tiles beside it.
//
// What bounds a small fill is the latency of a sweep's dependent steps, not
// its arithmetic (a 1024 x 1024 sweep is 5 us of VALU work on 256 CUs).  So:
//  - A halo value travels as one 64-bit word holding the angle and a tag
//    (launch epoch and sweep), stored and polled with relaxed device-scope
//    atomics: the word is its own flag, no fence, cache write-back or
//    invalidation stands between two sweeps, and the data arrives with the
//    poll that finds it.  Only colour 1 is exchanged: the ring's colour-0
//    sites are updated by every tile that reads them, to the same bits.
//  - The chain's per-sweep control needs its energy and accepted count:
//    every block stores its own sums in a word of its own and wave 0 of
//    every block reads those of the whole chain while the other waves poll
//    the halo (no atomic adds on one address).  Chains never wait for other
//    chains, and a block leaves when its chain is done.
//  - Equilibrium sweeps need no control: a tile waits for its neighbours'
//    halo only, after it has updated the colour-0 sites that do not need it,
//    so that a tile delayed by a double-precision decision delays its
//    neighbours and not the whole chain.
//  - The gap sites do not change: they are listed once per launch, and the
//    waves take the lists 64 entries at a time in turn.
// Two halo buffers alternate.  A tile that publishes sweep t + 2 has read
// its neighbours' sweep t + 1, which they published after reading its
// sweep t: the buffer it overwrites has been read.  The sums alternate
// between two words by the same argument over the whole chain.
// Measured, one chain with 100 states, whole fills, against the kernel this
// replaced (tiles written to memory and a device-wide barrier between
// sweeps): 64^2 4.4 us per sweep (8.5), 1024^2 8.5 us (18.9); 2048^2 28.7 us,
// against 41.3 us with one launch per sweep; four double-precision chains of
// 512^2 17.3 us, against two half-sweep launches of 12 us; 32 table chains of
// 256^2 17 us, against 38 us of half-sweeps and deferred redos.
//
// That a cooperative launch fits the GPU does not put all of its blocks on it:
// two blocks of 8 waves and 128 registers a lane need every register of a CU,
// in whole runs of 128, and a wave that came in beside another kernel's (of
// another thread's stream) may lie across two of them for as long as it
// stays.  So the blocks agree before they begin: each one counts itself, the
// last one lets the launch go, and a block that waits too long for that (2 ms)
// calls it off.  A launch called off leaves no trace, and its sweeps run one
// launch each.
//
// After that a block waits for running blocks only.  If it waits longer than
// its bound all the same (2 s unless the call sets another) it sets `abort`
// and every block leaves at its next wait; the host then reports an error.
// The update of a site is that of sweep_tile_kernel (or, for
// double-precision chains, of half_sweep_fp64_kernel), so the results are the
// same bit for bit.
struct ResidentCtl {
    // gen[0]: most sweeps any chain ran in this launch; gen[kResArrive]: blocks
    // on the GPU; gen[kResGoes]: 0 at launch, then kResGo or kResOff;
    // gen[kResStart]: the longest wait for that, in ticks.  (Behind one pointer:
    // the kernel has no scalar register left, and three more arguments cost up
    // to 5% of a sweep; as it is, agreeing costs 0.5 to 1.1%: us per sweep in
    // relaxation 9.91 and 10.01 at 1024^2, 20.7 and 20.9 at 2048^2.)
    unsigned int *gen;
    unsigned int *abort;           // nonzero: a block timed out
    unsigned long long *sums;      // [sweep parity][block]: energy | accepted << 46 | tag << 60, then
                                   // [block]: 1 once it has read its chain's state; zero at launch
    unsigned long long *halo;      // per block: colour 1 of even and odd sweeps, colour 0 at the start
    unsigned int *done_count;
    unsigned long long *work;
    float *states_out;             // recorded equilibrium states (nullable), their stride and K
    const int64_t *offsets;
    int64_t states_n_total;
    uint64_t wait_ticks;           // the longest wait, in ticks of the 100 MHz constant clock
    uint32_t epoch;                // launch tag of the halo words, << kResSweepBits
    int32_t count;                 // sweeps to run at most
    int32_t K;
};
constexpr uint64_t kPersistWaitTicks = 200000000ull;  // default wait bound: 2 s
constexpr uint32_t kPersistStartTicks = 200000u;      // default bound of the wait for the launch to go: 2 ms
constexpr int kResArrive = 1, kResGoes = 2, kResStart = 3;
constexpr unsigned int kResGo = 1u, kResOff = 2u;
constexpr int kResThreads = 512;
constexpr int kResWaves = kResThreads / 64;
constexpr int kResMaxBlocks = 512;  // blocks of a launch at most (8 sums words per lane of the reading wave)
constexpr int kResSweepBits = 13;   // sweeps_per_launch is at most 4096
constexpr uint32_t kResEpochs = 1u << (32 - kResSweepBits);
constexpr int kResMaxRows = 64;
// 64-bit words of a halo value and of one block's three halo buffers
template <typename RT> constexpr int res_words() { return (int)sizeof(RT) / 4; }
template <typename RT, int TH> constexpr int res_halo_len() { return 4 * kTileH + 2 * TH; }
template <typename RT, int TH> constexpr int res_halo_words() { return 3 * res_halo_len<RT, TH>() * res_words<RT>(); }

__device__ __forceinline__ void st_agent64(unsigned long long *p, unsigned long long v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bool fixed_rt(float v) { return is_fixed(v); }
__device__ __forceinline__ bool fixed_rt(double v) { return is_fixed_d(v); }

template <typename RT, int TH>
struct ResidentShared {
    static constexpr int N0 = TH * kTileH + 2 * kTileH + TH;  // colour-0 sites of the tile and its ring
    static constexpr int C0 = (N0 + 63) / 64;                 // 64-entry chunks of that list
    static constexpr int RCAP = (C0 + kResWaves - 1) / kResWaves * 64;
    // the equilibrium sums live in LDS where two blocks per CU leave room
    static constexpr bool ACC = TH * sizeof(RT) <= 128;
    alignas(16) RT a[2][TH + 4][kTileLS];
    alignas(16) RT acc[ACC ? 2 * TH : 1][kTileH];
    alignas(16) RT m2[ACC ? 2 * TH : 1][kTileH];
    uint16_t list0[C0 * 64];          // colour-0 gap sites: those that need no halo first; row << 7 | half-column
    uint16_t list1[TH * kTileH];      // colour 1: gap sites from the front, sampled sites from the back
    uint16_t redo[kResWaves][RCAP];   // sites of a wave's pass to be redone in double precision
    ChainState st;                    // this block's copy of its chain's state
    double w[kMaxFit];
    unsigned long long red_e[kResWaves];
    uint32_t red_a[kResWaves];
    int n0_inner, n0, n1, ns;
    int fail;
};

// A block counts itself (one thread); the last one lets the launch go.
__device__ __forceinline__ void res_arrive(unsigned int *gen)
{
    if (atomicAdd(gen + kResArrive, 1u) == gridDim.x - 1u) atomicCAS(gen + kResGoes, 0u, kResGo);
}

// Waits for the launch to go or calls it off (one thread); true if it goes.
__device__ __forceinline__ bool res_goes(unsigned int *gen)
{
    const uint64_t t0 = wall_clock64(), bound = ld_agent(gen + kResStart);
    unsigned int g = ld_agent(gen + kResGoes);
    while (g == 0u) {
        __builtin_amdgcn_s_sleep(1);
        if ((uint64_t)(wall_clock64() - t0) > bound) {
            g = atomicCAS(gen + kResGoes, 0u, kResOff);
            if (g == 0u) g = kResOff;
        } else {
            g = ld_agent(gen + kResGoes);
        }
    }
    return g == kResGo;
}

// One poll loop's bookkeeping: true when the wait must be given up.
__device__ __forceinline__ bool res_give_up(const ResidentCtl &rc, uint64_t t0, int n)
{
    __builtin_amdgcn_s_sleep(1);
    if ((n & 7) == 7 && ld_agent(rc.abort) != 0u) return true;
    if ((uint64_t)(wall_clock64() - t0) > rc.wait_ticks) {
        __hip_atomic_store(rc.abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    }
    return false;
}

// Waits for the halo value at p (res_words words tagged `tag`) and returns
// it in *out; false when the wait was given up.
__device__ __forceinline__ bool res_wait(const ResidentCtl &rc, const unsigned long long *p, uint32_t tag, float *out)
{
    unsigned long long v = ld_agent64(p);
    if ((uint32_t)(v >> 32) != tag) {
        const uint64_t t0 = wall_clock64();
        for (int n = 0;; ++n) {
            if (res_give_up(rc, t0, n)) return false;
            v = ld_agent64(p);
            if ((uint32_t)(v >> 32) == tag) break;
        }
    }
    *out = __uint_as_float((uint32_t)v);
    return true;
}

__device__ __forceinline__ bool res_wait(const ResidentCtl &rc, const unsigned long long *p, uint32_t tag, double *out)
{
    unsigned long long v = ld_agent64(p), w = ld_agent64(p + 1);
    if ((uint32_t)(v >> 32) != tag || (uint32_t)(w >> 32) != tag) {
        const uint64_t t0 = wall_clock64();
        for (int n = 0;; ++n) {
            if (res_give_up(rc, t0, n)) return false;
            v = ld_agent64(p);
            w = ld_agent64(p + 1);
            if ((uint32_t)(v >> 32) == tag && (uint32_t)(w >> 32) == tag) break;
        }
    }
    *out = __hiloint2double((int)(uint32_t)w, (int)(uint32_t)v);
    return true;
}

__device__ __forceinline__ void res_publish(unsigned long long *p, uint32_t tag, float v)
{
    st_agent64(p, ((unsigned long long)tag << 32) | __float_as_uint(v));
}

__device__ __forceinline__ void res_publish(unsigned long long *p, uint32_t tag, double v)
{
    st_agent64(p, ((unsigned long long)tag << 32) | (uint32_t)__double2loint(v));
    st_agent64(p + 1, ((unsigned long long)tag << 32) | (uint32_t)__double2hiint(v));
}

// The launch of one tile: block `slot` of the launch, block lb of the nblk
// blocks of chain cid.
template <typename RT, int TH, bool EDGE>
__device__ __forceinline__ void resident_tile(ResidentShared<RT, TH> &L, ChainState *states, const ChainDesc &d, int cid,
                                              int slot, int lb, int nblk, bool agree, const SweepConsts &sc,
                                              const CtlParams &cp, const ResidentCtl &rc)
{
    using RS = ResidentShared<RT, TH>;
    typedef RT v4 __attribute__((ext_vector_type(4)));
    constexpr bool F64 = sizeof(RT) == 8;
    constexpr int W = res_words<RT>();
    constexpr int HL = res_halo_len<RT, TH>() * W;  // words of one halo buffer
    constexpr int NQ = kTileH / 4;
    static_assert(4 * kTileH + 2 * TH + 4 <= kResThreads - 64, "one halo value per polling thread");
    const int tid = (int)threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nbx = d.S / kTileH, nby = nblk / nbx;
    const int ty = lb / nbx, tx = lb - ty * nbx;
    const int y0 = ty * TH, hx0 = tx * kTileH;
    if (agree) {
        if (tid == 0) L.fail = res_goes(rc.gen) ? 0 : 1;
        __syncthreads();
        if (L.fail) return;
    }
    const bool lead = lb == 0;  // the chain's first block
    RT *const h0p = (RT *)d.h[0], *const h1p = (RT *)d.h[1];
    RT *const acc0p = (RT *)d.acc[0], *const acc1p = (RT *)d.acc[1];
    RT *const m20p = (RT *)d.m2[0], *const m21p = (RT *)d.m2[1];

    // ---- the tile, its sums and its chain's state into LDS; the halo zero
    // (outside the grid: never a candidate nor a valid neighbour)
    for (int k = tid; k < 2 * (TH + 4) * kTileLS; k += kResThreads) {
        const int j = k % kTileLS, r = (k / kTileLS) % (TH + 4);
        if (r < 2 || r >= TH + 2 || j < 4 || j >= kTileH + 4) (&L.a[0][0][0])[k] = (RT)0;
    }
    for (int k = tid; k < 2 * TH * NQ; k += kResThreads) {
        const int cc = k / (TH * NQ), rr = (k / NQ) % TH, q = k % NQ, y = y0 + rr;
        v4 v = {(RT)0, (RT)0, (RT)0, (RT)0}, s = v, m = v;
        if (y < d.ny) {
            const int64_t idx = (int64_t)y * d.S + hx0 + 4 * q;
            v = *(const v4 *)((cc ? h1p : h0p) + idx);
            if (RS::ACC && acc0p) s = *(const v4 *)((cc ? acc1p : acc0p) + idx);
            if (RS::ACC && m20p) m = *(const v4 *)((cc ? m21p : m20p) + idx);
        }
        *(v4 *)&L.a[cc][rr + 2][4 + 4 * q] = v;
        if (RS::ACC) {
            *(v4 *)&L.acc[cc * TH + rr][4 * q] = s;
            *(v4 *)&L.m2[cc * TH + rr][4 * q] = m;
        }
    }
    {
        const unsigned long long *src = reinterpret_cast<const unsigned long long *>(states + cid);
        unsigned long long *dst = reinterpret_cast<unsigned long long *>(&L.st);
        for (int k = tid; k < (int)(sizeof(ChainState) / 8); k += kResThreads) dst[k] = src[k];
        for (int k = tid; k < kMaxFit; k += kResThreads) L.w[k] = cp.w[k];
    }
    if (tid == 0) {
        L.n0_inner = L.n0 = L.n1 = L.ns = 0;
        L.fail = 0;
    }
    __syncthreads();

    unsigned long long *const started = rc.sums + 2 * kResMaxBlocks + (slot - lb);
    if (tid == 0 && nblk > 1) st_agent64(started + lb, 1ull);

    // ---- halo exchange: a block's colour-1 buffer holds its rows 0, 1,
    // TH - 2 and TH - 1, then its first and last half-column; the colour-0
    // one rows 0 and TH - 1, then the columns
    unsigned long long *const mine = rc.halo + (int64_t)slot * 3 * HL;
    auto publish1 = [&](int buf, uint32_t tag) {
        for (int k = tid; k < 4 * kTileH + 2 * TH; k += kResThreads) {
            RT v;
            if (k < 4 * kTileH) {
                const int b = k / kTileH;
                v = L.a[1][b < 2 ? 2 + b : TH + b - 2][4 + k % kTileH];
            } else {
                const int b = k - 4 * kTileH;
                v = L.a[1][2 + (b < TH ? b : b - TH)][b < TH ? 4 : kTileH + 3];
            }
            res_publish(mine + buf * HL + k * W, tag, v);
        }
    };
    // the halo value this thread polls (threads of wave 0 poll none):
    // offset in the halo of the block that holds it, or -1, and its place
    int64_t src1 = -1, src0 = -1;
    int dst1 = 0, dst0 = 0;
    {
        const int up = ty > 0 ? slot - nbx : -1, dn = ty + 1 < nby ? slot + nbx : -1;
        const int w = tid - 64;
        int s = -1, o = 0, r = 0, j = 0;
        if (w < 0) {
        } else if (w < 2 * kTileH) {  // rows y0 - 1 and y0 - 2
            s = up, o = (w < kTileH ? 3 : 2) * kTileH + w % kTileH, r = w < kTileH ? 1 : 0, j = 4 + w % kTileH;
        } else if (w < 4 * kTileH) {  // rows y0 + TH and y0 + TH + 1
            s = dn, o = w - 2 * kTileH, r = w < 3 * kTileH ? TH + 2 : TH + 3, j = 4 + w % kTileH;
        } else if (w < 4 * kTileH + TH) {
            s = tx > 0 ? slot - 1 : -1, o = w + TH, r = 2 + w - 4 * kTileH, j = 3;
        } else if (w < 4 * kTileH + 2 * TH) {
            s = tx + 1 < nbx ? slot + 1 : -1, o = w - TH, r = 2 + w - 4 * kTileH - TH, j = kTileH + 4;
        } else if (w < 4 * kTileH + 2 * TH + 4) {  // corners
            const int k = w - 4 * kTileH - 2 * TH, b = k < 2 ? up : dn;
            const bool left = (k & 1) == 0;
            s = b >= 0 && (left ? tx > 0 : tx + 1 < nbx) ? b + (left ? -1 : 1) : -1;
            o = (k < 2 ? 3 : 0) * kTileH + (left ? kTileH - 1 : 0), r = k < 2 ? 1 : TH + 2, j = left ? 3 : kTileH + 4;
        }
        if (s >= 0) src1 = (int64_t)s * 3 * HL + o * W;
        dst1 = r * kTileLS + j;
        s = -1;
        if (w < 0) {
        } else if (w < kTileH) {
            s = up, o = kTileH + w, r = 1, j = 4 + w;
        } else if (w < 2 * kTileH) {
            s = dn, o = w - kTileH, r = TH + 2, j = 4 + w - kTileH;
        } else if (w < 2 * kTileH + TH) {
            s = tx > 0 ? slot - 1 : -1, o = w + TH, r = 2 + w - 2 * kTileH, j = 3;
        } else if (w < 2 * kTileH + 2 * TH) {
            s = tx + 1 < nbx ? slot + 1 : -1, o = w - TH, r = 2 + w - 2 * kTileH - TH, j = kTileH + 4;
        }
        if (s >= 0) src0 = (int64_t)s * 3 * HL + 2 * HL + o * W;
        dst0 = r * kTileLS + j;
    }
    auto wait1 = [&](int buf, uint32_t tag) {
        if (src1 < 0) return;
        RT v;
        if (res_wait(rc, rc.halo + src1 + buf * HL, tag, &v)) (&L.a[1][0][0])[dst1] = v;
        else L.fail = 1;
    };
    if (nblk > 1) {
        publish1(0, rc.epoch | 1u);
        for (int k = tid; k < 2 * kTileH + 2 * TH; k += kResThreads) {
            RT v;
            if (k < 2 * kTileH) {
                v = L.a[0][k < kTileH ? 2 : TH + 1][4 + k % kTileH];
            } else {
                const int b = k - 2 * kTileH;
                v = L.a[0][2 + (b < TH ? b : b - TH)][b < TH ? 4 : kTileH + 3];
            }
            res_publish(mine + 2 * HL + k * W, rc.epoch | 1u, v);
        }
        wait1(0, rc.epoch | 1u);
        if (src0 >= 0) {
            RT v;
            if (res_wait(rc, rc.halo + src0, rc.epoch | 1u, &v)) (&L.a[0][0][0])[dst0] = v;
            else L.fail = 1;
        }
        __syncthreads();
    }

    // ---- the lists: colour 0 in two rounds, first the gap sites whose
    // neighbours are all in the tile, then the others and the ring; colour 1
    // (a list's order does not matter: sites of a colour do not depend on
    // each other and the sums are integers)
    auto in_grid = [&](int c, int r, int j) {
        const int y = y0 - 2 + r, h = hx0 - 4 + j, s = (r + c) & 1;
        return !EDGE || (y >= 0 && y < d.ny && h >= 0 && h < ((d.nx - s + 1) >> 1));
    };
    auto append = [&](bool want, uint16_t *lst, int *n, int dir, uint16_t ent) {
        const uint64_t b = __ballot(want);
        int base = 0;
        if (lane == 0 && b) base = atomicAdd(n, (int)__popcll(b));
        base = __builtin_amdgcn_readfirstlane(base);
        if (want) lst[dir * (base + rank_below(b))] = ent;
    };
    for (int round = 0; round < 2; ++round) {
        for (int r = 2 + wid; r < TH + 2; r += kResWaves) {
            const int j = 4 + lane, s = r & 1;
            const bool inner = r > 2 && r < TH + 1 && (s ? j < kTileH + 3 : j > 4);
            append(inner == (round == 0) && in_grid(0, r, j) && !fixed_rt(L.a[0][r][j]), L.list0, &L.n0, 1,
                   (uint16_t)((r << 7) | j));
        }
        if (round == 0) {
            __syncthreads();
            if (tid == 0) L.n0_inner = L.n0;
            __syncthreads();
        } else {
            // the ring: the rows above and below, and in each row the one
            // colour-0 site beside the tile
            if (wid < 2) {
                const int r = wid ? TH + 2 : 1, j = 4 + lane;
                append(in_grid(0, r, j) && !fixed_rt(L.a[0][r][j]), L.list0, &L.n0, 1, (uint16_t)((r << 7) | j));
            }
            for (int k = wid; k * 64 < TH; k += kResWaves) {
                const int rr = k * 64 + lane, r = 2 + (rr < TH ? rr : 0), j = (r & 1) ? 3 : kTileH + 4;
                append(rr < TH && in_grid(0, r, j) && !fixed_rt(L.a[0][r][j]), L.list0, &L.n0, 1,
                       (uint16_t)((r << 7) | j));
            }
        }
    }
    for (int r = 2 + wid; r < TH + 2; r += kResWaves) {
        const int j = 4 + lane;
        const bool in = in_grid(1, r, j), gap = in && !fixed_rt(L.a[1][r][j]);
        append(gap, L.list1, &L.n1, 1, (uint16_t)((r << 7) | j));
        append(in && !gap, L.list1 + TH * kTileH - 1, &L.ns, -1, (uint16_t)((r << 7) | j));
    }
    __syncthreads();
    const int n0 = L.n0, n1 = L.n1, ns = L.ns, inner_chunks = L.n0_inner / 64;

    // ---- the sweeps
    int32_t phase = L.st.phase;
    bool due = false;  // a sweep was made whose control has not run
    int i = 0;
    for (;; ++i) {
        bool have = true;  // the halo of this sweep is in LDS
        if (due) {
            if (phase == PH_EQ) {
                // temperature and a stay as they are: the control's
                // divisions (1 us on one lane) wait until the chain is left,
                // unless the squared deviations need its 1 / k
                have = nblk == 1;
                if (tid == 0) {
                    if (L.st.eq_left > 1 && i < rc.count && !m20p) {
                        L.st.sweep += 1u;
                        L.st.eq_left -= 1;
                        if (lead) count_work(d, cp, rc.work);
                    } else {
                        L.st.e_fx = L.st.acc = 0ull;
                        control_core(L.st, d, cp, control_ratios(L.st, d, cp), lead ? rc.done_count : nullptr, lead ? rc.work : nullptr,
                                     [](uint32_t) { return 0.0; });
                    }
                }
            } else if (wid == 0) {
                // the chain's sums of the last sweep
                unsigned long long e = 0ull;
                uint32_t ac = 0u;
                if (nblk == 1) {
                    e = lane < kResWaves ? L.red_e[lane & (kResWaves - 1)] : 0ull;
                    ac = lane < kResWaves ? L.red_a[lane & (kResWaves - 1)] : 0u;
                } else {
                    const unsigned long long *p = rc.sums + (int64_t)((i - 1) & 1) * kResMaxBlocks + (slot - lb);
                    const uint32_t tag = (((uint32_t)(i - 1) >> 1) & 7u) + 1u;
                    unsigned long long v[kResMaxBlocks / 64];
#pragma unroll
                    for (int k = 0; k < kResMaxBlocks / 64; ++k)
                        v[k] = lane + 64 * k < nblk ? ld_agent64(p + lane + 64 * k) : (unsigned long long)tag << 60;
                    const uint64_t t0 = wall_clock64();
                    for (int n = 0;; ++n) {
                        bool ok = true;
#pragma unroll
                        for (int k = 0; k < kResMaxBlocks / 64; ++k) ok = ok && (uint32_t)(v[k] >> 60) == tag;
                        if (ok) break;
                        if (res_give_up(rc, t0, n)) {
                            L.fail = 1;
                            break;
                        }
#pragma unroll
                        for (int k = 0; k < kResMaxBlocks / 64; ++k)
                            if ((uint32_t)(v[k] >> 60) != tag) v[k] = ld_agent64(p + lane + 64 * k);
                    }
#pragma unroll
                    for (int k = 0; k < kResMaxBlocks / 64; ++k) {
                        e += v[k] & ((1ull << 46) - 1ull);
                        ac += (uint32_t)(v[k] >> 46) & 0x3FFFu;
                    }
                }
                wave_sum_63(e, ac);
                e = readlane64(e, 63);
                ac = (uint32_t)__builtin_amdgcn_readlane((int)ac, 63);
                const uint32_t t = L.st.sweep;
                // the control's three quotients by one division, a lane each
                const double num = lane == 0 ? (double)e * cp.e_unit : lane == 1 ? (double)(unsigned long long)ac : (double)(t + 1u);
                const double den = lane == 0 ? (double)d.ngp : lane == 1 ? (double)d.P : cp.k_a;
                const unsigned long long quo = (unsigned long long)__double_as_longlong(num / den);
                ControlRatios ratios;
                ratios.ope = __longlong_as_double((long long)readlane64(quo, 0));
                ratios.A = __longlong_as_double((long long)readlane64(quo, 1));
                ratios.ta = __longlong_as_double((long long)readlane64(quo, 2));
                double slope = 0.0;
                if (phase == PH_RELAX && t >= (uint32_t)cp.n_fit && t % (uint32_t)cp.n_f == 0u)
                    slope = ring_slope_wave(L.st.ring, ratios.ope, t, cp.n_fit, L.w, lane);
                if (lane == 0) {
                    control_core(L.st, d, cp, ratios, lead ? rc.done_count : nullptr, lead ? rc.work : nullptr,
                                 [&](uint32_t) { return slope; });
                }
            } else if (i < rc.count) {
                wait1(i & 1, rc.epoch | (uint32_t)(i + 1));
            }
            __syncthreads();
        }
        if (L.fail) break;
        phase = L.st.phase;
        if (phase == PH_DONE || i >= rc.count) break;
        const bool eq = phase == PH_EQ;
        const uint32_t sweep = L.st.sweep;
        unsigned long long e_thread = 0ull;
        uint32_t acc_thread = 0u;
        int n_redo = 0;
        // segment 0: the colour-0 chunks that need no halo, where it is still
        // under way; 1: the others; 2: colour 1.  Segment 0 is left out where
        // the halo is there, in floats and tiles of up to 32 rows only: elsewhere
        // that costs more than it saves (a relaxing sweep with it left out and
        // kept: 19.07 and 18.93 us for 4 chains of 512^2 doubles, 21.15 and
        // 21.00 us for 2048^2 floats).
        constexpr bool SKIP = !F64 && TH <= 32;
        const bool early = !SKIP || (eq && !have);
        for (int seg = early ? 0 : 1; seg < 3; ++seg) {
            const int c = seg == 2 ? 1 : 0;
            if (seg == 1 && !have) {
                wait1(i & 1, rc.epoch | (uint32_t)(i + 1));
                __syncthreads();
                if (L.fail) break;
            }
            const uint16_t *lst = c ? L.list1 : L.list0;
            const int n = c ? n1 : n0;
            const int k_end = seg == 0 ? inner_chunks : (n + 63) / 64;
            // wave w takes chunks w, w + kResWaves, ...; segment 1 goes on where 0 stopped
            int k = wid;
            if (seg == 1 && early) k += (inner_chunks > wid ? (inner_chunks - wid + kResWaves - 1) / kResWaves : 0) * kResWaves;
            for (; k < k_end; k += kResWaves) {
                const int e = k * 64 + lane;
                bool n64 = false;
                uint32_t ent = 0u;
                if (e < n) {
                    ent = lst[e];
                    const int r = (int)(ent >> 7), j = (int)(ent & 127u);
                    const int s = (r + c) & 1;  // y0 is even
                    const RT *oth = &L.a[c ^ 1][r][j];
                    const RT a0 = L.a[c][r][j];
                    const RT nL = fabs(oth[s - 1]), nR = fabs(oth[s]), nU = fabs(oth[-kTileLS]), nD = fabs(oth[kTileLS]);
                    const int y = y0 - 2 + r, h = hx0 - 4 + j;
                    uint32_t valid = 15u;
                    if (EDGE) {
                        const int Wo = (d.nx + s) >> 1;
                        valid = (h + s - 1 >= 0 ? 1u : 0u) | (h + s < Wo ? 2u : 0u) | (y > 0 ? 4u : 0u) |
                                (y + 1 < d.ny ? 8u : 0u);
                    }
                    const U4 ctr = {(uint32_t)y * (uint32_t)d.nx + (uint32_t)(2 * (h & ~1) + s), sweep, d.chain,
                                    d.image_id};
                    const U4 w = philox4x32_10(ctr, sc.seed_lo, sc.seed_hi);
                    const bool second = (h & 1) != 0;
                    const float u = unit24(second ? w.z : w.x), rr = unit24(second ? w.w : w.y);
                    const bool own = c == 1 || (r >= 2 && r < TH + 2 && j >= 4 && j < kTileH + 4);
                    if constexpr (F64) {
                        const SiteOutD o = update_site_d(a0, nL, nR, nU, nD, valid, (double)u, (double)rr, L.st.a_cur,
                                                         L.st.T, sc.q64, false);
                        L.a[c][r][j] = o.phi;
                        if (own) {
                            acc_thread += o.accepted ? 1u : 0u;
                            if (c == 1 && !eq) e_thread += energy_fx_d(o.e_bonds);
                        }
                    } else {
                        n64 = true;
                        const SiteOut o = update_site(a0, nL, nR, nU, nD, valid, u, rr, L.st.inv_T, L.st.dscale, false,
                                                      &n64);
                        if (!n64) {
                            L.a[c][r][j] = o.phi;
                            if (own) {
                                acc_thread += o.accepted ? 1u : 0u;
                                if (c == 1 && !eq) e_thread += energy_fx(o.e_bonds);
                            }
                        }
                    }
                }
                if constexpr (!F64) {  // too close to call: redone below
                    const uint64_t b = __ballot(n64);
                    if (b) {
                        if (n64) L.redo[wid][n_redo + rank_below(b)] = (uint16_t)ent;
                        n_redo += (int)__popcll(b);
                    }
                }
            }
            if (seg == 0) continue;
            // the wave's deferred decisions, in double precision from the same inputs
            if constexpr (!F64) {
                for (int e = lane; e < n_redo; e += 64) {
                    const uint32_t ent = L.redo[wid][e];
                    const int r = (int)(ent >> 7), j = (int)(ent & 127u);
                    const SiteOutD o = tile_redo_site(&L.a[0][0][0], TH + 4, c, r, j, y0, hx0, d.nx, d.ny, sweep, d.chain,
                                                      d.image_id, sc, 0, L.st.a_cur, L.st.T);
                    L.a[c][r][j] = (float)o.phi;
                    if (c == 1 || (r >= 2 && r < TH + 2 && j >= 4 && j < kTileH + 4)) {
                        acc_thread += o.accepted ? 1u : 0u;
                        if (c == 1 && !eq) e_thread += energy_fx((float)o.e_bonds);
                    }
                }
                n_redo = 0;
            }
            if (c == 1 && !eq) {
                // bond energies of the tile's sampled colour-1 sites
                for (int e = tid; e < ns; e += kResThreads) {
                    const uint32_t ent = L.list1[TH * kTileH - 1 - e];
                    const int r = (int)(ent >> 7), j = (int)(ent & 127u);
                    const int s = (r + 1) & 1;
                    const RT *oth = &L.a[0][r][j];
                    const RT nL = fabs(oth[s - 1]), nR = fabs(oth[s]), nU = fabs(oth[-kTileLS]), nD = fabs(oth[kTileLS]);
                    uint32_t valid = 15u;
                    if (EDGE) {
                        const int y = y0 - 2 + r, h = hx0 - 4 + j;
                        const int Wo = (d.nx + s) >> 1;
                        valid = (h + s - 1 >= 0 ? 1u : 0u) | (h + s < Wo ? 2u : 0u) | (y > 0 ? 4u : 0u) |
                                (y + 1 < d.ny ? 8u : 0u);
                    }
                    if constexpr (F64) e_thread += energy_fx_d(bond_energy_d(fabs(L.a[1][r][j]), nL, nR, nU, nD, valid, sc.q64));
                    else e_thread += energy_fx(bond_energy_half(0.5f * fabsf(L.a[1][r][j]), nL, nR, nU, nD, valid));
                }
                unsigned long long es = e_thread;
                uint32_t as = acc_thread;
                wave_sum_63(es, as);
                if (lane == 63) {
                    L.red_e[wid] = es;
                    L.red_a[wid] = as;
                }
            }
            __syncthreads();
        }
        if (L.fail) break;
        due = true;
        if (nblk > 1) {
            if (wid == 0 && !eq) {
                unsigned long long e = lane < kResWaves ? L.red_e[lane & (kResWaves - 1)] : 0ull;
                uint32_t a = lane < kResWaves ? L.red_a[lane & (kResWaves - 1)] : 0u;
                dpp_step<0x111, 0xF>(e, a);  // the sum over lanes 0 to 7 in lane 7
                dpp_step<0x112, 0xF>(e, a);
                dpp_step<0x114, 0xF>(e, a);
                const unsigned long long tag = (((uint32_t)i >> 1) & 7u) + 1u;
                if (lane == kResWaves - 1)
                    st_agent64(rc.sums + (int64_t)(i & 1) * kResMaxBlocks + slot,
                               e | ((unsigned long long)a << 46) | (tag << 60));
            }
            publish1((i + 1) & 1, rc.epoch | (uint32_t)(i + 2));
        }
        if (eq) {
            // the sweep's states into the equilibrium sums (the arithmetic of
            // accumulate_state), and recorded, while the halo is under way
            if (acc0p) {
                for (int k = tid; k < 2 * TH * NQ; k += kResThreads) {
                    const int cc = k / (TH * NQ), rr = (k / NQ) % TH, q = k % NQ, y = y0 + rr;
                    if (y >= d.ny) continue;
                    const int h = hx0 + 4 * q;
                    const int Wc = (d.nx - ((y + cc) & 1) + 1) >> 1;
                    const v4 v = *(const v4 *)&L.a[cc][rr + 2][4 + 4 * q];
                    const int64_t idx = (int64_t)y * d.S + h;
                    v4 *ap = RS::ACC ? (v4 *)&L.acc[RS::ACC ? cc * TH + rr : 0][4 * q] : (v4 *)((cc ? acc1p : acc0p) + idx);
                    v4 *mp = RS::ACC ? (v4 *)&L.m2[RS::ACC ? cc * TH + rr : 0][4 * q] : (v4 *)((cc ? m21p : m20p) + idx);
                    const v4 s0 = *ap;
                    v4 s1 = s0;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (!fixed_rt(v[e]) && h + e < Wc) s1[e] = s0[e] + v[e];
                    *ap = s1;
                    if (m20p) {
                        v4 m = *mp;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (!fixed_rt(v[e]) && h + e < Wc) {
                                if constexpr (F64)
                                    m[e] = fma(v[e] - s0[e] * L.st.inv_km1_d, v[e] - s1[e] * L.st.inv_k_d, m[e]);
                                else m[e] = fmaf(v[e] - s0[e] * L.st.inv_km1, v[e] - s1[e] * L.st.inv_k, m[e]);
                            }
                        *mp = m;
                    }
                }
            }
            if (rc.states_out) {
                const int64_t m = (int64_t)d.chain * rc.K + (rc.K - L.st.eq_left);
                float *o = rc.states_out + m * rc.states_n_total + rc.offsets[cid];
                for (int k = tid; k < TH * 2 * kTileH; k += kResThreads) {
                    const int rr = k / (2 * kTileH), xx = k % (2 * kTileH), y = y0 + rr, x = 2 * hx0 + xx;
                    if (y < d.ny && x < d.nx)
                        o[(int64_t)y * d.nx + x] = (float)fabs(L.a[(rr + xx) & 1][rr + 2][4 + (xx >> 1)]);
                }
            }
            __syncthreads();  // the state is read above, the control changes it
        }
    }
    // ---- the tile, its sums and the chain's state back to memory
    __syncthreads();
    if (L.fail) return;
    for (int k = tid; k < 2 * TH * NQ; k += kResThreads) {
        const int cc = k / (TH * NQ), rr = (k / NQ) % TH, q = k % NQ, y = y0 + rr;
        if (y >= d.ny) continue;
        const int64_t idx = (int64_t)y * d.S + hx0 + 4 * q;
        *(v4 *)((cc ? h1p : h0p) + idx) = *(const v4 *)&L.a[cc][rr + 2][4 + 4 * q];
        if (RS::ACC && acc0p) *(v4 *)((cc ? acc1p : acc0p) + idx) = *(const v4 *)&L.acc[RS::ACC ? cc * TH + rr : 0][4 * q];
        if (RS::ACC && m20p) *(v4 *)((cc ? m21p : m20p) + idx) = *(const v4 *)&L.m2[RS::ACC ? cc * TH + rr : 0][4 * q];
    }
    if (lead) {
        // once every block of the chain has read its state at the start
        // (equilibrium sweeps wait for the neighbours only)
        if (tid < nblk && nblk > 1) {
            const uint64_t t0 = wall_clock64();
            for (int n = 0; ld_agent64(started + tid) == 0ull; ++n)
                if (res_give_up(rc, t0, n)) break;
        }
        __syncthreads();
        const unsigned long long *src = reinterpret_cast<const unsigned long long *>(&L.st);
        unsigned long long *dst = reinterpret_cast<unsigned long long *>(states + cid);
        for (int k = tid; k < (int)(sizeof(ChainState) / 8); k += kResThreads) dst[k] = src[k];
        if (tid == 0) atomicMax(rc.gen, (unsigned int)i);
    }
}

template <typename RT, int TH>
__global__ __launch_bounds__(kResThreads) __attribute__((amdgpu_waves_per_eu(4))) void sweep_resident_kernel(
    const ChainDesc *descs, ChainState *states, BlockMap bm, SweepConsts sc, CtlParams cp, ResidentCtl rc)
{
    __shared__ ResidentShared<RT, TH> L;
    // the tile of this block (the XCD-aware order of sweep_tile_kernel)
    const uint32_t G = gridDim.x, b = blockIdx.x;
    const uint32_t per = G >> 3, rem = G & 7u, xcd = b & 7u;
    const int64_t slot = (int64_t)xcd * per + (int64_t)min(xcd, rem) + (int64_t)(b >> 3);
    const int k = find_chain(bm.start, bm.n, slot);
    const int lb = (int)(slot - bm.start[k]), nblk = (int)(bm.start[k + 1] - bm.start[k]);
    const int cid = bm.id[k];
    const ChainDesc d = descs[cid];
    const bool agree = (uint32_t)bm.n < G;  // a chain of several blocks: some wait for others
    if (agree && threadIdx.x == 0) res_arrive(rc.gen);
    if (states[cid].phase == PH_DONE) return;  // before this launch: no block of the chain starts
    const int nbx = d.S / kTileH;
    const int ty = lb / nbx, tx = lb - ty * nbx;
    const int y0 = ty * TH, hx0 = tx * kTileH;
    const bool edge = !(ty >= 1 && y0 + TH + 2 <= d.ny && tx >= 1 && hx0 + kTileH + 2 <= (d.nx >> 1));
    if (edge) resident_tile<RT, TH, true>(L, states, d, cid, (int)slot, lb, nblk, agree, sc, cp, rc);
    else resident_tile<RT, TH, false>(L, states, d, cid, (int)slot, lb, nblk, agree, sc, cp, rc);
}

// The double-precision sweep: the layout of half_sweep_body (a thread per
// pair of neighbouring sites of one half-row, one Philox call per pair) on
// half-grids of doubles, each site updated by update_site_d.  Every decision
// is final here, so nothing is deferred.  Bond energies are summed in fixed
// point of 2^-30.
template <bool DIAG, int ROWS>
__global__ __launch_bounds__(kBlock) void half_sweep_fp64_kernel(const ChainDesc *__restrict__ descs,
                                                                 ChainState *__restrict__ states,
                                                                 BlockMap bm,
                                                                 int colour, SweepConsts sc, int or_only,
                                                                 uint8_t *__restrict__ flags)
{
    constexpr int PX = kBlock / ROWS;
    int lb;
    const int c = chain_of_block(bm, (int64_t)blockIdx.x, &lb);
    ChainState *stp = states + c;
    const int phase = stp->phase;
    if (phase == PH_DONE) return;
    const ChainDesc d = descs[c];
    const int nbx = ((d.S >> 1) + PX - 1) / PX;
    const int by = lb / nbx;
    const int bx = lb - by * nbx;
    const int y = by * ROWS + (int)(threadIdx.x / PX);
    const int h0 = 2 * (bx * PX + (int)(threadIdx.x % PX));
    const uint32_t sweep = stp->sweep;
    const double T = stp->T, a = stp->a_cur;
    const bool want_energy = (colour == 1) && (phase != PH_EQ);
    const bool want_acc = phase != PH_EQ;
    unsigned long long e_thread = 0ull;
    uint32_t acc_thread = 0u;

    if (y < d.ny) {
        const int s = (y + colour) & 1;
        const int W = (d.nx - s + 1) >> 1;
        const int Wo = (d.nx + s) >> 1;
        if (h0 < W) {
            const bool two = (h0 + 1) < W;
            double *mine = (double *)(colour ? d.h[1] : d.h[0]) + (int64_t)y * d.S;
            const double *oth = (const double *)(colour ? d.h[0] : d.h[1]) + (int64_t)y * d.S;
            const bool vL = h0 + s - 1 >= 0, vM = h0 + s < Wo, vR = h0 + s + 1 < Wo;
            const bool vU = y > 0, vD = y + 1 < d.ny;
            const double2 v = gldd2(mine + h0);
            const double oL = fabs(gldd(oth + max(h0 + s - 1, 0)));
            const double oM = fabs(gldd(oth + h0 + s));
            const double oR = fabs(gldd(oth + min(h0 + s + 1, d.S - 1)));
            const double2 up = gldd2(oth + (vU ? -(int64_t)d.S : 0) + h0);
            const double2 dn = gldd2(oth + (vD ? (int64_t)d.S : 0) + h0);
            const bool fixed0 = is_fixed_d(v.x), fixed1 = !two || is_fixed_d(v.y);
            double u0 = 0.5, r0 = 0.5, u1 = 0.5, r1 = 0.5;
            if (!or_only && (!fixed0 || !fixed1)) {
                const U4 ctr = {(uint32_t)y * (uint32_t)d.nx + (uint32_t)(2 * h0 + s), sweep, d.chain, d.image_id};
                const U4 w = philox4x32_10(ctr, sc.seed_lo, sc.seed_hi);
                u0 = (double)unit24(w.x);
                r0 = (double)unit24(w.y);
                u1 = (double)unit24(w.z);
                r1 = (double)unit24(w.w);
            }
            const uint32_t val0 = (vL ? 1u : 0u) | (vM ? 2u : 0u) | (vU ? 4u : 0u) | (vD ? 8u : 0u);
            const uint32_t val1 = 1u | (vR ? 2u : 0u) | (vU ? 4u : 0u) | (vD ? 8u : 0u);
            const SiteOutD o0 = update_site_d(fabs(v.x), oL, oM, fabs(up.x), fabs(dn.x), val0, u0, r0, a, T,
                                              sc.q64, or_only != 0);
            const SiteOutD o1 = update_site_d(fabs(v.y), oM, oR, fabs(up.y), fabs(dn.y), val1, u1, r1, a, T,
                                              sc.q64, or_only != 0);
            const bool w0 = !fixed0, w1 = two && !fixed1;
            const double out0 = w0 ? o0.phi : v.x;
            const double out1 = w1 ? o1.phi : v.y;
            if (two) gstd2(mine + h0, make_double2(out0, out1));
            else if (w0) gstd(mine + h0, out0);
            double *accp = (double *)(colour ? d.acc[1] : d.acc[0]);
            if (phase == PH_EQ && accp) {
                double *acc = accp + (int64_t)y * d.S;
                double *m2p = (double *)(colour ? d.m2[1] : d.m2[0]);
                double *m2 = m2p ? m2p + (int64_t)y * d.S : nullptr;
                const double ik = stp->inv_k_d, ikm1 = stp->inv_km1_d;
                if (w0) accumulate_state_d(acc + h0, m2 ? m2 + h0 : nullptr, out0, ik, ikm1);
                if (w1) accumulate_state_d(acc + h0 + 1, m2 ? m2 + h0 + 1 : nullptr, out1, ik, ikm1);
            }
            acc_thread = (w0 && o0.accepted ? 1u : 0u) + (w1 && o1.accepted ? 1u : 0u);
            if (want_energy)
                e_thread = energy_fx_d(fixed0 ? o0.e_before : o0.e_bonds) +
                           (!two ? 0ull : energy_fx_d(fixed1 ? o1.e_before : o1.e_bonds));
            if (DIAG && flags) {
                const int64_t x0 = 2 * h0 + s;
                if (w0) flags[(int64_t)y * d.nx + x0] = (uint8_t)o0.flags;
                if (w1) flags[(int64_t)y * d.nx + x0 + 2] = (uint8_t)o1.flags;
            }
        }
    }
    if (!want_acc) return;
    // block sums: a thread's energy is below 2^34 and its count at most 2,
    // so 64-bit lane sums hold both (count in the top 8 bits)
    unsigned long long sum = e_thread | ((unsigned long long)acc_thread << 56);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    __shared__ unsigned long long red[kBlock / 64];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long e = 0ull, n = 0ull;
        for (int i = 0; i < kBlock / 64; ++i) {
            e += red[i] & 0x00FFFFFFFFFFFFFFull;
            n += red[i] >> 56;
        }
        if (e) atomicAdd(&stp->e_fx, e);
        if (n) atomicAdd(&stp->acc, n);
    }
}

// The double-precision sweep with the gap sites compacted onto consecutive
// lanes: the list building of half_sweep_compact_body (1024 sites per block,
// CR half-rows, two site pairs per thread, the pair's Philox words drawn in
// pass 1) on double half-grids, each listed gap site updated by
// update_site_d and each sampled site of colour 1 given its bond energy by
// bond_energy_d when the sweep's energy is wanted.  Per site the arithmetic
// is that of half_sweep_fp64_kernel, so the results are bit-identical to it.
template <bool DIAG, int CR>
__global__ __launch_bounds__(kBlock) void half_sweep_fp64_compact_kernel(const ChainDesc *__restrict__ descs,
                                                                         ChainState *__restrict__ states,
                                                                         BlockMap bm, int colour, SweepConsts sc,
                                                                         int or_only, uint8_t *__restrict__ flags)
{
    constexpr int PPR = kCompactSites / CR / 2;  // site pairs per block row
    constexpr int NW = kBlock / 64;
    __shared__ uint2 gap_list[kCompactSites];  // as in half_sweep_compact_body
    __shared__ uint16_t fixed_list[kCompactSites];
    __shared__ uint32_t wave_count[2][2][NW];
    __shared__ unsigned long long red[NW];

    int lb;
    const int c = chain_of_block(bm, (int64_t)blockIdx.x, &lb);
    ChainState *stp = states + c;
    const int phase = stp->phase;
    if (phase == PH_DONE) return;
    const ChainDesc d = descs[c];
    const int nbx = ((d.S >> 1) + PPR - 1) / PPR;
    const int by = lb / nbx;
    const int bx = lb - by * nbx;
    const uint32_t sweep = stp->sweep;
    const double T = stp->T, a_cur = stp->a_cur;
    const bool want_energy = (colour == 1) && (phase != PH_EQ);
    const bool want_acc = phase != PH_EQ;
    double *const mine = (double *)(colour ? d.h[1] : d.h[0]);
    const double *const oth = (const double *)(colour ? d.h[0] : d.h[1]);
    double *const accp = (phase == PH_EQ) ? (double *)(colour ? d.acc[1] : d.acc[0]) : nullptr;
    double *const m2p = accp ? (double *)(colour ? d.m2[1] : d.m2[0]) : nullptr;

    // pass 1: pairs t and t + 256 of the block, both read first
    bool gap[2][2], fix[2][2];
    uint32_t wu[2][2], wr[2][2];
    double2 pv[2];
    bool in[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int pi = (int)threadIdx.x + j * kBlock;
        const int y = by * CR + pi / PPR;
        const int h0 = 2 * (bx * PPR + pi % PPR);
        const int s = (y + colour) & 1;
        in[j] = y < d.ny && h0 < ((d.nx - s + 1) >> 1);
        // rows and pairs outside the grid read pair 0 of row 0 instead
        pv[j] = gldd2(mine + (in[j] ? (int64_t)y * d.S + h0 : 0));
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int pi = (int)threadIdx.x + j * kBlock;
        const int y = by * CR + pi / PPR;
        const int h0 = 2 * (bx * PPR + pi % PPR);
        const int s = (y + colour) & 1;
        const bool two = in[j] && (h0 + 1) < ((d.nx - s + 1) >> 1);
        gap[j][0] = in[j] && !is_fixed_d(pv[j].x);
        gap[j][1] = two && !is_fixed_d(pv[j].y);
        fix[j][0] = want_energy && in[j] && !gap[j][0];
        fix[j][1] = want_energy && two && !gap[j][1];
        wu[j][0] = wu[j][1] = wr[j][0] = wr[j][1] = 0u;
        if (!or_only && (gap[j][0] || gap[j][1])) {
            const U4 ctr = {(uint32_t)y * (uint32_t)d.nx + (uint32_t)(2 * h0 + s), sweep, d.chain, d.image_id};
            const U4 w = philox4x32_10(ctr, sc.seed_lo, sc.seed_hi);
            wu[j][0] = w.x;
            wr[j][0] = w.y;
            wu[j][1] = w.z;
            wr[j][1] = w.w;
        }
    }
    const int lane = (int)(threadIdx.x & 63), wid = (int)(threadIdx.x >> 6);
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint32_t pre[2][2] = {{0u, 0u}, {0u, 0u}};
#pragma unroll
    for (int L = 0; L < 2; ++L) {
        if (L == 1 && !want_energy) continue;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint64_t b0 = __ballot(L ? fix[j][0] : gap[j][0]);
            const uint64_t b1 = __ballot(L ? fix[j][1] : gap[j][1]);
            pre[L][j] = (uint32_t)(__popcll(b0 & below) + __popcll(b1 & below));
            if (lane == 0) wave_count[L][j][wid] = (uint32_t)(__popcll(b0) + __popcll(b1));
        }
    }
    __syncthreads();
    int n_list[2] = {0, 0};
#pragma unroll
    for (int L = 0; L < 2; ++L) {
        if (L == 1 && !want_energy) continue;
        uint32_t base0 = 0u, base1 = 0u, tot0 = 0u, tot1 = 0u;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const uint32_t c0 = wave_count[L][0][w], c1 = wave_count[L][1][w];
            base0 += (w < wid) ? c0 : 0u;
            base1 += (w < wid) ? c1 : 0u;
            tot0 += c0;
            tot1 += c1;
        }
        n_list[L] = (int)(tot0 + tot1);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            uint32_t pos = (j ? tot0 + base1 : base0) + pre[L][j];
            const uint32_t pi = threadIdx.x + (uint32_t)j * kBlock;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const uint32_t idx = 2u * pi + (uint32_t)k;
                if (L == 0 && gap[j][k]) {
                    gap_list[pos] = make_uint2((wu[j][k] & 0xFFFFFF00u) | (idx & 0xFFu),
                                               (wr[j][k] & 0xFFFFFF00u) | (idx >> 8));
                    ++pos;
                }
                if (L == 1 && fix[j][k]) {
                    fixed_list[pos] = (uint16_t)idx;
                    ++pos;
                }
            }
        }
    }
    __syncthreads();

    // a listed site: row, half-row position, colour offset, valid neighbours,
    // and its four neighbours (loaded from clamped positions when missing)
    auto locate = [&](uint32_t idx, int &y, int &h, int &s, uint32_t &valid) {
        const int pi = (int)(idx >> 1);
        y = by * CR + pi / PPR;
        h = 2 * (bx * PPR + pi % PPR) + (int)(idx & 1u);
        s = (y + colour) & 1;
        const int Wo = (d.nx + s) >> 1;
        valid = (h + s - 1 >= 0 ? 1u : 0u) | (h + s < Wo ? 2u : 0u) | (y > 0 ? 4u : 0u) | (y + 1 < d.ny ? 8u : 0u);
    };
    auto neighbours = [&](int y, int h, int s, uint32_t valid, double &nL, double &nR, double &nU, double &nD) {
        const double *orow = oth + (int64_t)y * d.S;
        nL = fabs(gldd(orow + max(h + s - 1, 0)));
        nR = fabs(gldd(orow + min(h + s, d.S - 1)));
        nU = fabs(gldd(orow + ((valid & 4u) ? -(int64_t)d.S : 0) + h));
        nD = fabs(gldd(orow + ((valid & 8u) ? (int64_t)d.S : 0) + h));
    };

    // a thread takes at most 4 gap and 4 sampled sites, each below 2^33 in
    // energy units: the energy stays below 2^44 over a block, the count
    // (at most 1024) rides in the top 12 bits
    unsigned long long e_thread = 0ull;
    uint32_t acc_thread = 0u;
    // pass 2: the listed gap sites.  Unrolled over a thread's at most four
    // entries: in a loop the compiler keeps the double update's constants in
    // registers across iterations (~116 VGPRs, 4 waves per SIMD); unrolled,
    // the kernel takes 50 (8 waves)
#pragma unroll
    for (int k = 0; k < kCompactSites / kBlock; ++k) {
        const int i = (int)threadIdx.x + k * kBlock;
        if (i >= n_list[0]) break;
        const uint2 e = gap_list[i];
        int y, h, s;
        uint32_t valid;
        locate((e.x & 0xFFu) | ((e.y & 0xFFu) << 8), y, h, s, valid);
        double nL, nR, nU, nD;
        neighbours(y, h, s, valid, nL, nR, nU, nD);
        double *sp = mine + (int64_t)y * d.S + h;
        const double a = fabs(gldd(sp));
        // the low 8 bits of each word hold the index; unit24 uses the top 24
        const double u = or_only ? 0.5 : (double)unit24(e.x);
        const double r = or_only ? 0.5 : (double)unit24(e.y);
        const SiteOutD o = update_site_d(a, nL, nR, nU, nD, valid, u, r, a_cur, T, sc.q64, or_only != 0);
        gstd(sp, o.phi);
        if (accp)
            accumulate_state_d(accp + (int64_t)y * d.S + h, m2p ? m2p + (int64_t)y * d.S + h : nullptr, o.phi,
                               stp->inv_k_d, stp->inv_km1_d);
        acc_thread += o.accepted ? 1u : 0u;
        if (want_energy) e_thread += energy_fx_d(o.e_bonds);
        if (DIAG && flags) flags[(int64_t)y * d.nx + 2 * h + s] = (uint8_t)o.flags;
    }
    // pass 3: bond energies of the sampled sites of colour 1
#pragma unroll
    for (int k = 0; k < kCompactSites / kBlock; ++k) {
        const int i = (int)threadIdx.x + k * kBlock;
        if (i >= n_list[1]) break;
        int y, h, s;
        uint32_t valid;
        locate((uint32_t)fixed_list[i], y, h, s, valid);
        double nL, nR, nU, nD;
        neighbours(y, h, s, valid, nL, nR, nU, nD);
        const double a = fabs(gldd(mine + (int64_t)y * d.S + h));
        e_thread += energy_fx_d(bond_energy_d(a, nL, nR, nU, nD, valid, sc.q64));
    }
    if (!want_acc) return;
    unsigned long long sum = e_thread | ((unsigned long long)acc_thread << 52);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    if (lane == 0) red[wid] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long e = 0ull, n = 0ull;
        for (int i = 0; i < NW; ++i) {
            e += red[i] & 0x000FFFFFFFFFFFFFull;
            n += red[i] >> 52;
        }
        if (e) atomicAdd(&stp->e_fx, e);
        if (n) atomicAdd(&stp->acc, n);
    }
}

// control_chain for every chain, one thread per chain.  With `swap` (after
// a fused tile sweep, which read h and wrote h2) it first exchanges h and h2
// of every chain that sweep updated (those not done), toggling the chain's
// `swapped` flag; with `control` 0 it does only that.
__global__ void control_kernel(ChainDesc *__restrict__ descs, ChainState *__restrict__ states, int n,
                               CtlParams cp, unsigned int *done_count, unsigned long long *work, int swap,
                               int control)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    if (swap && states[c].phase != PH_DONE) {
        ChainDesc &d = descs[c];
        float *t0 = d.h[0], *t1 = d.h[1];
        d.h[0] = d.h2[0];
        d.h[1] = d.h2[1];
        d.h2[0] = t0;
        d.h2[1] = t1;
        states[c].swapped ^= 1;
    }
    if (control) control_chain(descs, states, c, cp, done_count, work);
}

// Zeroes the control words given (null: skipped) and n64 64-bit words at
// `wide`, in one launch of one block: the counters and control words a run of
// sweeps starts from (one small kernel in place of a memset per word).
__global__ void clear_words_kernel(unsigned int *w0, unsigned int *w1, unsigned int *w2,
                                   unsigned long long *wide, int n64)
{
    const int t = (int)threadIdx.x;
    if (t == 0) {
        if (w0) *w0 = 0u;
        if (w1) *w1 = 0u;
        if (w2) *w2 = 0u;
    }
    for (int k = t; k < n64; k += (int)blockDim.x) wide[k] = 0ull;
}

// The control words a resident launch starts from: its four words at gen and
// n64 zeros at `sums`.
__global__ void clear_resident_kernel(unsigned int *gen, uint32_t start_ticks, unsigned long long *sums, int n64)
{
    const int t = (int)threadIdx.x;
    if (t < 4) gen[t] = t == kResStart ? start_ticks : 0u;
    for (int k = t; k < n64; k += (int)blockDim.x) sums[k] = 0ull;
}

// Zeroes the halo words of the resident sweeps.
__global__ void clear_halo_kernel(unsigned long long *w, int64_t n)
{
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x)
        w[k] = 0ull;
}

// 1 for every chain that is done, else 0 (for rebuilding the launch list).
__global__ void done_flags_kernel(const ChainState *__restrict__ states, int n, uint8_t *__restrict__ out)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < n) out[c] = states[c].phase == PH_DONE ? 1 : 0;
}

// phi_sum at every site of image blockIdx.y: sum over its R chains of the
// equilibrium sums (K > 1) or the final states (K == 1).  With phi_m2, also
// the sum over the R K states of the squared deviation from their mean: two
// passes over the R final states (K == 1), or the chains' own sums combined
// with the spread of their means (Chan et al.'s pairwise rule, K > 1).
__global__ void finalize_kernel(const ChainDesc *__restrict__ descs, ImgArgs imgs, int R,
                                int K, const uint8_t *__restrict__ sampled, float *__restrict__ phi_sum,
                                float *__restrict__ phi_m2)
{
    const ImgDev im = imgs.at((int)blockIdx.y);
    const int64_t n = (int64_t)im.nx * im.ny;
    const ChainDesc *dc = descs + (int64_t)blockIdx.y * R;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        float s = 0.0f, q = 0.0f;
        if (!sampled[im.offset + i] && K > 0) {
            const int y = (int)(i / im.nx);
            const int x = (int)(i - (int64_t)y * im.nx);
            const int c = (x + y) & 1;
            const int64_t j = (int64_t)y * dc[0].S + (x >> 1);
            for (int r = 0; r < R; ++r) s += (K > 1) ? dc[r].acc[c][j] : angle_of(dc[r].h[c][j]);
            if (phi_m2) {
                const float mean = s / (float)(R * K);
                for (int r = 0; r < R; ++r) {
                    const float d = ((K > 1) ? dc[r].acc[c][j] / (float)K : angle_of(dc[r].h[c][j])) - mean;
                    q = fmaf((float)K * d, d, q);
                    if (K > 1) q += dc[r].m2[c][j];
                }
            }
        }
        phi_sum[im.offset + i] = s;
        if (phi_m2) phi_m2[im.offset + i] = q;
    }
}

// finalize_kernel for double-precision chains: the same sums taken in
// double and rounded once.
__global__ void finalize_fp64_kernel(const ChainDesc *__restrict__ descs, ImgArgs imgs, int R,
                                     int K, const uint8_t *__restrict__ sampled, float *__restrict__ phi_sum,
                                     float *__restrict__ phi_m2)
{
    const ImgDev im = imgs.at((int)blockIdx.y);
    const int64_t n = (int64_t)im.nx * im.ny;
    const ChainDesc *dc = descs + (int64_t)blockIdx.y * R;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        double s = 0.0, q = 0.0;
        if (!sampled[im.offset + i] && K > 0) {
            const int y = (int)(i / im.nx);
            const int x = (int)(i - (int64_t)y * im.nx);
            const int c = (x + y) & 1;
            const int64_t j = (int64_t)y * dc[0].S + (x >> 1);
            for (int r = 0; r < R; ++r)
                s += (K > 1) ? ((const double *)dc[r].acc[c])[j] : fabs(((const double *)dc[r].h[c])[j]);
            if (phi_m2) {
                const double mean = s / (double)(R * K);
                for (int r = 0; r < R; ++r) {
                    const double dv = ((K > 1) ? ((const double *)dc[r].acc[c])[j] / (double)K
                                               : fabs(((const double *)dc[r].h[c])[j])) - mean;
                    q = fma((double)K * dv, dv, q);
                    if (K > 1) q += ((const double *)dc[r].m2[c])[j];
                }
            }
        }
        phi_sum[im.offset + i] = (float)s;
        if (phi_m2) phi_m2[im.offset + i] = (float)q;
    }
}

// Records the current states of the listed chains that are in their
// equilibrium phase (after both half-sweeps of an equilibrium sweep, before
// the control kernel counts it): state r K + k of chain r after its k-th
// equilibrium sweep goes to out[(r K + k) n_total + offset + i], row-major
// over the image's sites (samples included).  `segs` blocks per listed chain.
__global__ void record_states_kernel(const ChainDesc *__restrict__ descs, const ChainState *__restrict__ states,
                                     const int64_t *__restrict__ offsets, const int32_t *__restrict__ ids,
                                     int segs, int K, int fp64, int64_t n_total, float *__restrict__ out)
{
    const int c = ids[blockIdx.x / segs];
    const ChainState *stp = states + c;
    if (stp->phase != PH_EQ) return;
    const ChainDesc d = descs[c];
    const int64_t n = (int64_t)d.nx * d.ny;
    const int64_t m = (int64_t)d.chain * K + (K - stp->eq_left);
    float *o = out + m * n_total + offsets[c];
    const int seg = (int)(blockIdx.x % segs);
    for (int64_t i = (int64_t)seg * blockDim.x + threadIdx.x; i < n; i += (int64_t)segs * blockDim.x) {
        const int y = (int)(i / d.nx);
        const int x = (int)(i - (int64_t)y * d.nx);
        const int64_t j = (int64_t)y * d.S + (x >> 1);
        const float *hp = ((x + y) & 1) ? d.h[1] : d.h[0];
        o[i] = fp64 ? (float)fabs(((const double *)hp)[j]) : angle_of(hp[j]);
    }
}

constexpr int kMaxQuantileStates = 256;

// The sampled sites kept for fitting when a fraction `hold` of them is held
// out for validation: a sample is held out when the uniform of its site,
// word 0 of Philox4x32-10 with counter (y nx + x, 0xFFFFFFFE, 0, 0x40000000)
// and the seed as key, is below `hold`.
constexpr uint32_t kHoldoutSweep = 0xFFFFFFFEu;
constexpr uint32_t kHoldoutStream = 0x40000000u;

__global__ void holdout_kernel(int nx, int ny, const uint8_t *__restrict__ sampled, uint32_t seed_lo,
                               uint32_t seed_hi, double hold, uint8_t *__restrict__ fit)
{
    const int64_t n = (int64_t)nx * ny;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        uint8_t keep = 0;
        if (sampled[i]) {
            const U4 w = philox4x32_10(U4{(uint32_t)i, kHoldoutSweep, 0u, kHoldoutStream}, seed_lo, seed_hi);
            keep = (double)unit24(w.x) < hold ? 0 : 1;
        }
        fit[i] = keep;
    }
}

// Partial sums of |z - z_hat| and counts over the held-out samples
// (sampled but not kept for fitting), one pair per block.
__global__ void holdout_error_kernel(int64_t n, const float *__restrict__ z, const uint8_t *__restrict__ sampled,
                                     const uint8_t *__restrict__ fit, const float *__restrict__ z_hat,
                                     double *__restrict__ psum, unsigned long long *__restrict__ pcount)
{
    double s = 0.0;
    unsigned long long c = 0ull;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        if (sampled[i] && !fit[i]) {
            s += fabs((double)z[i] - (double)z_hat[i]);
            ++c;
        }
    for (int off = 32; off > 0; off >>= 1) {
        s += __shfl_xor(s, off);
        c += __shfl_xor(c, off);
    }
    __shared__ double ss[kBlock / 64];
    __shared__ unsigned long long sc[kBlock / 64];
    if ((threadIdx.x & 63) == 0) {
        ss[threadIdx.x >> 6] = s;
        sc[threadIdx.x >> 6] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kBlock / 64; ++i) {
            ss[0] += ss[i];
            sc[0] += sc[i];
        }
        psum[blockIdx.x] = ss[0];
        pcount[blockIdx.x] = sc[0];
    }
}

// Sorts v[0..N-1] ascending with Batcher's odd-even merge sort, a fixed
// network of compare-exchanges: with N a compile-time constant and every loop
// unrolled, all indices are constants, so v stays in registers.
template <int N>
__device__ __forceinline__ void odd_even_merge_sort(float (&v)[N])
{
#pragma unroll
    for (int p = 1; p < N; p <<= 1)
#pragma unroll
        for (int k = p; k >= 1; k >>= 1)
#pragma unroll
            for (int j = k % p; j + k < N; j += 2 * k)
#pragma unroll
                for (int i = 0; i < k; ++i)
                    if (i + j + k < N && (i + j) / (2 * p) == (i + j + k) / (2 * p)) {
                        const float a = v[i + j], b = v[i + j + k];
                        v[i + j] = fminf(a, b);
                        v[i + j + k] = fmaxf(a, b);
                    }
}

// A bitonic sequence v[0..N-1], N a power of two, sorted ascending.
template <int N>
__device__ __forceinline__ void bitonic_merge(float (&v)[N])
{
#pragma unroll
    for (int k = N / 2; k >= 1; k >>= 1)
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (!(i & k)) {
                const float a = v[i], b = v[i + k];
                v[i] = fminf(a, b);
                v[i + k] = fmaxf(a, b);
            }
}

// v[a] and v[a + 1] (if there is one) for a wave-uniform a, without putting
// v in memory: the eight entries around a by a branch (in a large v), one of
// them by selects.
template <int N>
__device__ __forceinline__ void pick_two(const float (&v)[N], int a, float &va, float &vb)
{
    va = vb = 0.0f;
#pragma unroll
    for (int g = 0; g < N; g += 8)
        if (N <= 32 || (a & ~7) == g) {
            if (N > 32) __asm__ volatile("");
#pragma unroll
            for (int m = g; m < g + 8 && m < N; ++m) {
                va = m == a ? v[m] : va;
                if (m + 1 < N) vb = m == a ? v[m + 1] : vb;
            }
        }
}

// States first, first + 1, ... of element i into v, +inf beyond state M - 1
// (state M - 1 is read again there, so that every load is issued at once);
// at least `sure` of them exist.
template <int N>
__device__ __forceinline__ void load_states(float (&v)[N], const float *src, int first, int sure, int M,
                                            int64_t n_total, uint32_t i)
{
    src += (int64_t)first * n_total;
#pragma unroll
    for (int m = 0; m < N; ++m) {
        // (opaque, so that the addresses of many rows are not held in registers at once)
        if (N > 32) __asm__ volatile("" : "+s"(src));
        v[m] = gldi(src, i);
        src += m + 1 < sure || first + m + 1 < M ? n_total : 0;
    }
#pragma unroll
    for (int m = 0; m < N; ++m)
        if (m >= sure) v[m] = first + m < M ? v[m] : INFINITY;
}

// The p-quantile from the order statistics around h = (M - 1) p, a = floor(h),
// back-transformed like the mean (double precision, rounded once).
__device__ __forceinline__ float quantile_value(double h, int a, int M, float va, float vb, double lo, double hi)
{
#pragma clang fp contract(off)
    const double phi_p = a >= M - 1 ? (double)va : (double)va + (h - (double)a) * ((double)vb - (double)va);
    const double tt = phi_p / kTwoPi;
    return (float)(lo * (1.0 - tt) + hi * tt);
}

// Quantiles of the M realizations (states[m n_total + site]) at each gap site
// of image blockIdx.y; sampled sites get their data value.  A wave works along
// `span` sites: it lists their gap sites in LDS, 256 sites at a time, and
// whenever 64 are listed each lane sorts the states of one of them in
// registers, so that no lane idles over a sample; waves do not wait for each
// other.  The network is that of the next multiple of eight entries (states
// beyond M are +inf and sort last).  With BIG (M > 128, N = 128) two runs of N
// states are sorted one after the other, the first kept in LDS meanwhile;
// their lower and upper halves (minima and maxima of one run against the other
// reversed) are bitonic and are merged in turn.  Bound by reading the states,
// with the comparisons next (2300 min/max for M = 100); 2048^2 sites, half of
// them gaps, three quantiles, a whole call: M = 100 475 us (939 with a sort of
// 128 entries at every site), M = 50 246 us (336), M = 16 99 us (104); 1024^2
// sites, M = 200: 0.35 ms (48 ms with an insertion sort in LDS).
// waves per SIMD that the registers of a network leave
constexpr int quantile_waves(int n, bool big) { return big ? 1 : n <= 48 ? 8 : n <= 104 ? 4 : 3; }
// Up to 32 states a lane takes each site as it comes: reading the states
// bounds such a sort even with half of the lanes idle (M = 16, half gaps: 99
// us a call, 117 with the list).
constexpr bool quantile_lists(int n) { return n > 32; }
template <int N, bool BIG>
__global__ __launch_bounds__(BIG ? 64 : kBlock)
__attribute__((amdgpu_waves_per_eu(quantile_waves(N, BIG)))) void quantile_kernel(
    ImgArgs imgs, RangeArgs range, ProbArgs probs, int nq, const float *__restrict__ z, const uint8_t *__restrict__ sampled, const float *__restrict__ st, int M,
    int64_t n_total, int64_t span, float *__restrict__ out)
{
    constexpr int NW = BIG ? 1 : kBlock / 64;
    constexpr bool LIST = quantile_lists(N);
    constexpr int GROUP = LIST ? 256 : 64;  // sites at a time
    __shared__ uint32_t lists[NW][LIST ? GROUP + 64 : 1];
    __shared__ float runs[BIG ? N * 64 : 1];
    const ImgDev im = imgs.at((int)blockIdx.y);
    const int64_t n = (int64_t)im.nx * im.ny;
    const double lo = range.lo((int)blockIdx.y), hi = range.hi((int)blockIdx.y);
    const int lane = (int)(threadIdx.x & 63), wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t first = ((int64_t)blockIdx.x * NW + wid) * span;
    if (first >= n) return;
    const int64_t k0 = im.offset + first;
    const uint32_t len = (uint32_t)min(n - first, span);
    uint32_t *list = lists[wid];
    int listed = 0;
    // the quantiles of this lane's site
    auto site = [&](uint32_t i) {
        float v[N];
        load_states<N>(v, st + k0, 0, BIG ? N : N - 8, M, n_total, i);
        odd_even_merge_sort<N>(v);
        if constexpr (BIG) {
            float *run = runs + lane;
#pragma unroll
            for (int m = 0; m < N; ++m) run[m * 64] = v[m];
            load_states<N>(v, st + k0, N, 0, M, n_total, i);
            odd_even_merge_sort<N>(v);
#pragma unroll
            for (int m = 0; m < N; ++m) {
                const float x = run[(N - 1 - m) * 64];
                run[(N - 1 - m) * 64] = fmaxf(v[m], x);
                v[m] = fminf(v[m], x);
            }
            bitonic_merge<N>(v);
            // the lower half to LDS, the upper one from there
#pragma unroll
            for (int m = 0; m < N; ++m) {
                const float x = run[m * 64];
                run[m * 64] = v[m];
                v[m] = x;
            }
            bitonic_merge<N>(v);
        }
        for (int q = 0; q < nq; ++q) {
            const double h = (double)(M - 1) * probs.v[q];
            const int a = __builtin_amdgcn_readfirstlane((int)floor(h));
            float va, vb;
            if (BIG && a < N) {
                va = runs[a * 64 + lane];
                vb = a + 1 < N ? runs[(a + 1) * 64 + lane] : v[0];
            } else {
                pick_two<N>(v, BIG ? a - N : a, va, vb);
            }
            out[q * n_total + k0 + i] = quantile_value(h, a, M, va, vb, lo, hi);
        }
    };
    for (uint32_t g = 0; g < len; g += GROUP) {
        uint8_t smp[GROUP / 64];
#pragma unroll
        for (int r = 0; r < GROUP / 64; ++r) {
            const uint32_t i = g + 64u * r + (uint32_t)lane;
            smp[r] = sampled[k0 + min(i, len - 1u)];
        }
#pragma unroll
        for (int r = 0; r < GROUP / 64; ++r) {
            const uint32_t i = g + 64u * r + (uint32_t)lane;
            const bool gap = i < len && !smp[r];
            if (LIST) {
                const uint64_t b = __ballot(gap);
                if (gap) list[listed + rank_below(b)] = i;
                listed += (int)__popcll(b);
            } else if (gap) {
                site(i);
            }
            if (i < len && !gap)
                for (int q = 0; q < nq; ++q) out[q * n_total + k0 + i] = z[k0 + i];
        }
        if (!LIST) continue;
        __builtin_amdgcn_wave_barrier();
        const bool last = g + GROUP >= len;
        while (listed >= 64 || (last && listed > 0)) {
            // the last listed sites (those before them stay listed)
            const int take = min(listed, 64);
            listed -= take;
            if (lane < take) site(list[listed + lane]);
            __builtin_amdgcn_wave_barrier();
        }
    }
}

template <int N, bool BIG>
void launch_quantiles(hipStream_t stream, int64_t max_sites, int n, const ImgArgs &imgs, const RangeArgs &range,
                      const ProbArgs &probs, int nq, const float *z, const uint8_t *sampled, const float *states, int M,
                      int64_t n_total, float *z_q)
{
    // four times as many waves as the 1024 SIMDs hold at once (one for BIG),
    // each along at least 64 sites: at M = 100, half gaps, one to sixteen
    // times as many take 511, 494, 481 and 506 us
    const int64_t waves = 1024 * quantile_waves(N, BIG) * (BIG ? 1 : 4);
    const int64_t span = std::max<int64_t>(64, ((max_sites * n + waves - 1) / waves + 63) / 64 * 64);
    const int64_t per_block = span * (BIG ? 1 : kBlock / 64);
    hipLaunchKernelGGL((quantile_kernel<N, BIG>), dim3((unsigned)((max_sites + per_block - 1) / per_block), n),
                       dim3(BIG ? 64 : kBlock), 0, stream, imgs, range, probs, nq, z, sampled, states, M, n_total, span,
                       z_q);
}

// Spread of the prediction: the standard deviation over the M realizations
// of z = G^{-1}(phi), which is (z_max - z_min) / (2 pi) times that of phi,
// sqrt(m2 / (M - 1)); zero at sampled sites and for M = 1.
__global__ void spread_kernel(ImgArgs imgs, RangeArgs range, int M,
                              const uint8_t *__restrict__ sampled, const float *__restrict__ phi_m2,
                              float *__restrict__ z_std)
{
    const ImgDev im = imgs.at((int)blockIdx.y);
    const int64_t n = (int64_t)im.nx * im.ny;
    const double scale = (range.hi((int)blockIdx.y) - range.lo((int)blockIdx.y)) / kTwoPi;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t k = im.offset + i;
        float v = 0.0f;
        if (!sampled[k] && M > 1) v = (float)(scale * sqrt(fmax((double)phi_m2[k], 0.0) / (double)(M - 1)));
        z_std[k] = v;
    }
}

// Half-grids of one double-precision chain back to a full row-major grid.
__global__ void unsplit_fp64_kernel(const ChainDesc *__restrict__ descs, double *__restrict__ phi)
{
    const ChainDesc d = descs[0];
    const int64_t n = (int64_t)d.nx * d.ny;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int y = (int)(i / d.nx);
        const int x = (int)(i - (int64_t)y * d.nx);
        const double *hp = (const double *)(((x + y) & 1) ? d.h[1] : d.h[0]);
        phi[i] = fabs(hp[(int64_t)y * d.S + (x >> 1)]);
    }
}

// Half-grids of one chain back to a full row-major grid of angles.
__global__ void unsplit_kernel(const ChainDesc *__restrict__ descs, float *__restrict__ phi)
{
    const ChainDesc d = descs[0];
    const int64_t n = (int64_t)d.nx * d.ny;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int y = (int)(i / d.nx);
        const int x = (int)(i - (int64_t)y * d.nx);
        const float *hp = ((x + y) & 1) ? d.h[1] : d.h[0];
        phi[i] = angle_of(hp[(int64_t)y * d.S + (x >> 1)]);
    }
}

// Energy of a full grid of angles as the sweep accumulates it.
__global__ void grid_energy_kernel(const float *__restrict__ phi, int nx, int ny, float q,
                                   unsigned long long *out)
{
    unsigned long long e = 0ull;
    const int64_t n = (int64_t)nx * ny;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int y = (int)(i / nx);
        const int x = (int)(i - (int64_t)y * nx);
        if (((x + y) & 1) != 1) continue;
        float nb[4] = {0.f, 0.f, 0.f, 0.f};
        uint32_t valid = 0u;
        if (x > 0) { nb[0] = phi[i - 1]; valid |= 1u; }
        if (x + 1 < nx) { nb[1] = phi[i + 1]; valid |= 2u; }
        if (y > 0) { nb[2] = phi[i - nx]; valid |= 4u; }
        if (y + 1 < ny) { nb[3] = phi[i + nx]; valid |= 8u; }
        e += energy_fx(site_energy(phi[i], nb, valid, q));
    }
    for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off);
    if ((threadIdx.x & 63) == 0 && e) atomicAdd(out, e);
}

// Per-block min / max / count of the sampled values of image blockIdx.y.
__global__ void map_minmax_kernel(ImgArgs imgs, const float *__restrict__ z,
                                  const uint8_t *__restrict__ sampled, float *__restrict__ pmin,
                                  float *__restrict__ pmax, unsigned long long *__restrict__ pcount,
                                  unsigned int *__restrict__ pbad)
{
    const ImgDev im = imgs.at((int)blockIdx.y);
    const int64_t n = (int64_t)im.nx * im.ny;
    float lo = INFINITY, hi = -INFINITY;
    unsigned long long cnt = 0ull;
    unsigned int bad = 0u;
    // four sites a round, their loads issued together (a 64^2 image is one
    // round of four blocks)
    const int64_t nt = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += 4 * nt) {
        uint8_t m[4];
        float v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t j = im.offset + min(i + k * nt, n - 1);
            m[k] = sampled[j];
            v[k] = z[j];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (i + k * nt >= n || !m[k]) continue;
            if (!isfinite(v[k])) {
                bad = 1u;
                continue;
            }
            lo = fminf(lo, v[k]);
            hi = fmaxf(hi, v[k]);
            ++cnt;
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, off));
        hi = fmaxf(hi, __shfl_xor(hi, off));
        cnt += __shfl_xor(cnt, off);
        bad |= __shfl_xor(bad, off);
    }
    __shared__ float slo[kBlock / 64], shi[kBlock / 64];
    __shared__ unsigned long long scnt[kBlock / 64];
    __shared__ unsigned int sbad[kBlock / 64];
    const int wid = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        slo[wid] = lo;
        shi[wid] = hi;
        scnt[wid] = cnt;
        sbad[wid] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kBlock / 64; ++i) {
            slo[0] = fminf(slo[0], slo[i]);
            shi[0] = fmaxf(shi[0], shi[i]);
            scnt[0] += scnt[i];
            sbad[0] |= sbad[i];
        }
        const int64_t k = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
        pmin[k] = slo[0];
        pmax[k] = shi[0];
        pcount[k] = scnt[0];
        pbad[k] = sbad[0];
    }
}

// The map of image blockIdx.y from its range; with `parts` > 0 (one image) the
// range is first reduced from that many partial results, by every block for
// itself, written to `found` (host memory: minimum, maximum, samples, whether
// one is not finite), and nothing is mapped unless it is valid.
__global__ __launch_bounds__(kBlock) void map_apply_kernel(ImgArgs imgs, RangeArgs range, int parts,
                                                           const float *__restrict__ pmin,
                                                           const float *__restrict__ pmax,
                                                           const unsigned long long *__restrict__ pcount,
                                                           const unsigned int *__restrict__ pbad,
                                                           double *__restrict__ found, const float *__restrict__ z,
                                                           const uint8_t *__restrict__ sampled,
                                                           float *__restrict__ phi)
{
#pragma clang fp contract(off)
    const ImgDev im = imgs.at((int)blockIdx.y);
    double zmin, zmax;
    if (parts > 0) {
        __shared__ float slo[kBlock / 64], shi[kBlock / 64];
        __shared__ uint32_t scnt[kBlock / 64], sbad[kBlock / 64];
        float lo = INFINITY, hi = -INFINITY;
        uint32_t cnt = 0u, bad = 0u;
        for (int k = (int)threadIdx.x; k < parts; k += kBlock) {
            lo = fminf(lo, pmin[k]);
            hi = fmaxf(hi, pmax[k]);
            cnt = min(cnt + (uint32_t)min(pcount[k], 2ull), 2u);  // fewer than two samples are refused
            bad |= pbad[k];
        }
        for (int off = 32; off > 0; off >>= 1) {
            lo = fminf(lo, __shfl_xor(lo, off));
            hi = fmaxf(hi, __shfl_xor(hi, off));
            cnt += __shfl_xor(cnt, off);
            bad |= __shfl_xor(bad, off);
        }
        if ((threadIdx.x & 63) == 0) {
            slo[threadIdx.x >> 6] = lo;
            shi[threadIdx.x >> 6] = hi;
            scnt[threadIdx.x >> 6] = cnt;
            sbad[threadIdx.x >> 6] = bad;
        }
        __syncthreads();
        lo = slo[0], hi = shi[0], cnt = scnt[0], bad = sbad[0];
        for (int k = 1; k < kBlock / 64; ++k) {
            lo = fminf(lo, slo[k]);
            hi = fmaxf(hi, shi[k]);
            cnt += scnt[k];
            bad |= sbad[k];
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            found[0] = (double)lo;
            found[1] = (double)hi;
            found[2] = (double)cnt;
            found[3] = (double)bad;
        }
        if (bad || cnt < 2u || !(hi > lo)) return;
        zmin = (double)lo;
        zmax = (double)hi;
    } else {
        zmin = range.lo((int)blockIdx.y);
        zmax = range.hi((int)blockIdx.y);
    }
    const int64_t n = (int64_t)im.nx * im.ny;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t j = im.offset + i;
        phi[j] = sampled[j] ? (float)(kTwoPi * (((double)z[j] - zmin) / (zmax - zmin))) : 0.0f;
    }
}

__global__ void predict_kernel(ImgArgs imgs, RangeArgs range, int M,
                               const float *__restrict__ z, const uint8_t *__restrict__ sampled,
                               const float *__restrict__ phi_sum, float *__restrict__ z_hat)
{
#pragma clang fp contract(off)
    const ImgDev im = imgs.at((int)blockIdx.y);
    const double zmin = range.lo((int)blockIdx.y), zmax = range.hi((int)blockIdx.y);
    const int64_t n = (int64_t)im.nx * im.ny;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t j = im.offset + i;
        if (sampled[j]) {
            z_hat[j] = z[j];
        } else {
            const double t = ((double)phi_sum[j] / (double)M) / kTwoPi;
            z_hat[j] = (float)(zmin * (1.0 - t) + zmax * t);
        }
    }
}

// Partial-result blocks of an image of n sites: one per 4096 sites, at most
// kMapBlocks.  A function of the image alone, so that an image's e_s (a sum
// of doubles) does not depend on the batch it is in.
__host__ __device__ inline int image_blocks(int64_t n)
{
    const int64_t b = (n + 4095) / 4096;
    return (int)(b < 1 ? 1 : (b > kMapBlocks ? kMapBlocks : b));
}

// The same for exact results (minima, maxima, counts): one per 1024 sites.
int minmax_blocks(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + 1023) / 1024, kMapBlocks)); }

// Per-block sums of -cos(q (phi_i - phi_j)) over sample-sample bonds.  Thread t
// < 256 of a block adds its sites' terms in a fixed order, site by site, the
// right bond before the lower one.  The cosines bound the kernel (in double,
// and a 64^2 image has one block), so 1024 threads evaluate them, four sites
// each, into LDS, and 256 of them add up 16 sites' terms (zeros where there is
// no bond): 64^2 21 us before, 12 now; 1024^2 30, 14.
constexpr int kEsThreads = 1024;
__global__ __launch_bounds__(kEsThreads) void sample_energy_kernel(ImgArgs imgs, const float *__restrict__ phi,
                                                                   const uint8_t *__restrict__ sampled, double q,
                                                                   double *__restrict__ psum,
                                                                   unsigned long long *__restrict__ pcount)
{
    constexpr int SITES = 16 * kBlock;  // sites of a round
    __shared__ double term[2][SITES];
    __shared__ double ss[kBlock / 64];
    __shared__ unsigned int sc[kEsThreads / 64];
    const ImgDev im = imgs.at((int)blockIdx.y);
    const int64_t n = (int64_t)im.nx * im.ny;
    const int nbk = image_blocks(n);  // this image's blocks (the grid covers the largest image)
    if ((int)blockIdx.x >= nbk) return;
    const int tid = (int)threadIdx.x;
    double s = 0.0;
    unsigned int cnt = 0u;
    // step k of thread t: site (k nbk + block) kBlock + t
    const int64_t first = (int64_t)blockIdx.x * kBlock, stride = (int64_t)nbk * kBlock;
    for (int64_t k0 = 0; first + k0 * stride < n; k0 += SITES / kBlock) {
        for (int k = tid >> 8; k < SITES / kBlock; k += kEsThreads / kBlock) {
            const int64_t i = first + (k0 + k) * stride + (tid & (kBlock - 1));
            double right = 0.0, below = 0.0;
            if (i < n && sampled[im.offset + i]) {
                const int64_t j = im.offset + i;
                const int y = (int)(i / im.nx);
                const int x = (int)(i - (int64_t)y * im.nx);
                const double a = (double)phi[j];
                if (x + 1 < im.nx && sampled[j + 1]) {
                    right = cos(q * (a - (double)phi[j + 1]));
                    ++cnt;
                }
                if (y + 1 < im.ny && sampled[j + im.nx]) {
                    below = cos(q * (a - (double)phi[j + im.nx]));
                    ++cnt;
                }
            }
            term[0][k * kBlock + (tid & (kBlock - 1))] = right;
            term[1][k * kBlock + (tid & (kBlock - 1))] = below;
        }
        __syncthreads();
        if (tid < kBlock)
#pragma unroll
            for (int k = 0; k < SITES / kBlock; ++k) {
                s -= term[0][k * kBlock + tid];
                s -= term[1][k * kBlock + tid];
            }
        __syncthreads();
    }
    for (int off = 32; off > 0; off >>= 1) {
        s += __shfl_xor(s, off);
        cnt += __shfl_xor(cnt, off);
    }
    const int wid = tid >> 6;
    if ((tid & 63) == 0) {
        if (wid < kBlock / 64) ss[wid] = s;
        sc[wid] = cnt;
    }
    __syncthreads();
    if (tid == 0) {
        unsigned long long c = sc[0];
        for (int i = 1; i < kBlock / 64; ++i) ss[0] += ss[i];
        for (int i = 1; i < kEsThreads / 64; ++i) c += sc[i];
        const int64_t k = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
        psum[k] = ss[0];
        pcount[k] = c;
    }
}

__global__ void philox_kernel(const uint32_t *__restrict__ ctr, uint32_t k0, uint32_t k1, int64_t n,
                              uint32_t *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    U4 c = {ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3]};
    const U4 w = philox4x32_10(c, k0, k1);
    out[4 * i] = w.x;
    out[4 * i + 1] = w.y;
    out[4 * i + 2] = w.z;
    out[4 * i + 3] = w.w;
}

// Plain copy of n 16-byte words: the calibration probe for HBM byte counters.
__global__ void copy_probe_kernel(const float4 *__restrict__ src, float4 *__restrict__ dst, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

__global__ void ring_slope_kernel(const double *e, int n, CtlParams cp, double *out)
{
    double ring[kMaxFit];
    for (int j = 0; j < n; ++j) ring[j] = e[j];
    // values e[0..n-1] sit in ring slots 0..n-1, i.e. the newest is at t = n-1
    *out = ring_slope(ring, (uint32_t)(n - 1), n, cp.w);
}

// ====================================================================== host

struct mpr_ctx {
    int device = 0;
    std::string err;
    void *scratch = nullptr;          // small device scratch (partials, counters)
    void *static_ws = nullptr;        // this device's static_workspace (device address)
    // pinned host memory: the first kHostWordsBytes mirror the scratch's
    // control words (done counter, sweeps run, abort word); the
    // rest stages small read-backs (the per-block partials of the map and
    // of the sample energies) in one copy each
    unsigned int *done_host = nullptr;
    // blocks of the resident sweep kernel that the device holds at once, by
    // tile rows and angle bytes (0: no cooperative launch on this device)
    std::map<std::pair<int, int>, int64_t> persist_cap;
    uint32_t halo_epoch = 0;          // resident launches since the halo words were cleared; 0: not cleared yet
    // sweeps of one launch and less run on a context-owned stream (captured
    // into HIP graphs), ordered after and before the caller's with two events
    hipStream_t gstream = nullptr;
    hipEvent_t ev_in = nullptr, ev_out = nullptr, ev_t0 = nullptr, ev_t1 = nullptr;
    // tuned block shape by what the cost of a sweep depends on: type and
    // options, chains, largest sides, blocks (all chains together) and share of
    // gaps (shapes before `next` are timed; a run too short to time them all
    // goes on in the next call)
    struct Tuned {
        int next = 0, best = -1;
        float ms = 0.0f;
    };
    std::map<std::tuple<int, int, int, int, int64_t, int>, Tuned> tuned_rows;
    // profiling
    bool profile = false;
    double prof_ms = 0.0;
    int64_t prof_launches = 0;
    int32_t last_tile = 0;
    // e(T, L) tables: key -> (1 + e) per temperature
    std::map<std::tuple<int, int, double, int, double, double, int, int, double, double, uint64_t>,
             std::vector<double>>
        tables;
};

// Records an error text on the context (also used by the network kernels' host code).
int mpr_set_error(mpr_ctx *ctx, int code, const char *msg)
{
    if (ctx) ctx->err = msg;
    return code;
}

// Checks the device pointers of a call (name, pointer; null ones are
// skipped, the callers test the required ones first): each must be device
// memory of the context's device, or managed memory.  A host pointer would
// otherwise reach a kernel and fault the GPU.  Returns MPR_OK, or
// MPR_ERR_ARG with an error text naming the argument.
int mpr_check_device(mpr_ctx *ctx, const char *call,
                     std::initializer_list<std::pair<const char *, const void *>> ptrs)
{
    for (const auto &np : ptrs) {
        if (!np.second) continue;
        hipPointerAttribute_t a;
        std::memset(&a, 0, sizeof a);
        const hipError_t e = hipPointerGetAttributes(&a, np.second);
        if (e != hipSuccess) (void)hipGetLastError();  // not an address HIP knows: clear the error
        const bool managed = a.isManaged || a.type == hipMemoryTypeManaged || a.type == hipMemoryTypeUnified;
        if (e != hipSuccess || !(managed || (a.type == hipMemoryTypeDevice && a.device == ctx->device))) {
            char buf[256];
            snprintf(buf, sizeof buf, "%s: %s is not device memory of device %d", call, np.first, ctx->device);
            return mpr_set_error(ctx, MPR_ERR_ARG, buf);
        }
    }
    return MPR_OK;
}

namespace {

int fail(mpr_ctx *ctx, int code, const char *fmt, ...)
{
    if (ctx) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        ctx->err = buf;
    }
    return code;
}

#define HIP_TRY(ctx, expr)                                                                              \
    do {                                                                                                \
        hipError_t e_ = (expr);                                                                         \
        if (e_ != hipSuccess) return fail((ctx), MPR_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

int64_t round_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

int half_stride(int nx) { return (int)round_up((nx + 1) / 2, 64); }

// Bytes of one half-grid of `eb`-byte angles.
int64_t half_grid_bytes(int nx, int ny, int eb = 4) { return (int64_t)ny * half_stride(nx) * eb; }

// Host memory for a read-back of `bytes`: the context's pinned staging
// area when it fits, else `spill` (pageable), resized.
char *stage_for(mpr_ctx *ctx, int64_t bytes, std::vector<char> &spill)
{
    if (bytes <= kHostStageBytes - kHostWordsBytes) return (char *)ctx->done_host + kHostWordsBytes;
    spill.resize((size_t)bytes);
    return spill.data();
}

// The images of a call (and, where given, their ranges) as kernel arguments;
// more than kArgImages of them are copied to d_img and d_zmm, from `hi`, which
// the caller keeps until it has waited for the stream.
int image_args(mpr_ctx *ctx, hipStream_t stream, const mpr_image *imgs, int n, std::vector<ImgDev> &hi, ImgDev *d_img,
               ImgArgs &out)
{
    hi.resize(n);
    for (int b = 0; b < n; ++b) hi[b] = {imgs[b].offset, imgs[b].nx, imgs[b].ny};
    std::memset(&out, 0, sizeof out);
    if (n <= kArgImages) {
        for (int b = 0; b < n; ++b) out.own[b] = hi[b];
    } else {
        HIP_TRY(ctx, hipMemcpyAsync(d_img, hi.data(), n * sizeof(ImgDev), hipMemcpyHostToDevice, stream));
        out.dev = d_img;
    }
    return MPR_OK;
}

int range_args(mpr_ctx *ctx, hipStream_t stream, const double *zmin_zmax, int n, double *d_zmm, RangeArgs &out)
{
    std::memset(&out, 0, sizeof out);
    if (n <= kArgImages) {
        std::memcpy(out.own, zmin_zmax, (size_t)n * 16);
    } else {
        HIP_TRY(ctx, hipMemcpyAsync(d_zmm, zmin_zmax, (size_t)n * 16, hipMemcpyHostToDevice, stream));
        out.dev = d_zmm;
    }
    return MPR_OK;
}

// Simple bump allocator over the caller's workspace.
struct Carver {
    char *base;
    int64_t cap, used = 0;
    void *take(int64_t bytes)
    {
        used = round_up(used, 256);
        if (used + bytes > cap) return nullptr;
        void *p = base + used;
        used += bytes;
        return p;
    }
};

// Sweep block shapes: half-rows per block, and whether gap sites are
// compacted onto lanes (1024 sites per block) or not (512 sites per block);
// or a fused tile sweep (a whole sweep per launch on tiles of `rows` rows x
// 2 kTileH columns, single precision only).
struct Shape {
    int rows;
    bool compact;
    bool fused;
    bool persist;  // fused sweeps, many per cooperative launch (sweep_resident_kernel)
};
// The last two are not values of mpr_params.tile_rows: they are the resident
// shapes of chains whose 32-row tiles the GPU does not hold at once.
constexpr int kNumShapes = 20;
constexpr int kNumParamShapes = 18;
constexpr int kNumPlainShapes = 4;
constexpr int kNumUnfusedShapes = 7;   // the shapes of double-precision chains
constexpr Shape kShapes[kNumShapes] = {{1, false, false}, {2, false, false}, {4, false, false}, {8, false, false},
                                       {2, true, false},  {4, true, false},  {8, true, false},
                                       {16, false, true}, {24, false, true}, {32, false, true},
                                       {48, false, true}, {8, false, true},  {12, false, true},
                                       {8, false, true, true},  {12, false, true, true}, {16, false, true, true},
                                       {24, false, true, true}, {32, false, true, true},
                                       {48, false, true, true}, {kResMaxRows, false, true, true}};
// Block prefix sums are kept once for every number of tile rows: the
// resident shapes of 8 to 48 rows share those of the fused shapes, and the
// 64-row one takes the place of the 8-row one.
constexpr int kNumStarts = 18;
constexpr int start_of(int k)
{
    constexpr int same[kNumShapes] = {0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 11, 12, 7, 8, 9, 10, 13};
    return same[k];
}
constexpr int kDefaultShape = 2;  // plain, 4 half-rows
constexpr int kSmallTileShape = 11;  // fused, 8 rows: its blocks measure a chain set
static_assert(kShapes[kSmallTileShape].fused && kShapes[kSmallTileShape].rows == 8, "8-row tiles");

int tile_code(const Shape &sh)
{
    return (sh.persist ? std::min(sh.rows, 32) : sh.rows) | (sh.compact ? MPR_TILE_COMPACT : 0) | (sh.fused ? MPR_TILE_FUSED : 0) |
           (sh.persist ? MPR_TILE_PERSIST : 0);
}

// Shape index of a tile_rows value (rows | MPR_TILE_COMPACT, MPR_TILE_FUSED or
// MPR_TILE_FUSED | MPR_TILE_PERSIST), or -1.
int shape_of(int tile)
{
    for (int k = 0; k < kNumParamShapes; ++k)
        if (tile == tile_code(kShapes[k])) return k;
    return -1;
}

// Sweep blocks of one chain (half-row stride S, ny rows) for block shape k.
int64_t shape_blocks(int S, int ny, int k)
{
    const Shape sh = kShapes[k];
    if (sh.fused) return (int64_t)(S / kTileH) * ((ny + sh.rows - 1) / sh.rows);
    const int px = sh.compact ? kCompactSites / sh.rows / 2 : kBlock / sh.rows;  // site pairs per block row
    return (int64_t)((S / 2 + px - 1) / px) * ((ny + sh.rows - 1) / sh.rows);
}

int64_t chain_blocks(const ChainDesc &d, int k) { return shape_blocks(d.S, d.ny, k); }

// Mask words per sweep block of shape k (one bit per site of the block).
int redo_words(int k) { return kShapes[k].fused ? 0 : (kShapes[k].compact ? kCompactSites : 2 * kBlock) / 32; }

// Workspace bytes of the deferred-redo buffers for `chains` chains of an
// nx x ny grid (an upper bound over every block shape).
int64_t redo_bytes(int nx, int ny, int64_t chains)
{
    int64_t words = 0, blocks = 0;
    for (int k = 0; k < kNumShapes; ++k) {
        const int64_t b = shape_blocks(half_stride(nx), ny, k);
        words = std::max(words, b * redo_words(k));
        blocks = std::max(blocks, b);
    }
    return chains * (words * 4 + blocks / 8 + 8) + 1024;
}

bool valid_params(const mpr_params *p)
{
    // q = 1/2 (the paper's value) runs on either sweep; 0 < q < 1/2 on the
    // double-precision one (the single-precision kernels are written for 1/2)
    return p && (p->q == 0.5 || (p->q > 0.0 && p->q < 0.5 && p->fp64 == 1)) && p->R >= 1 && p->K >= 0 &&
           p->n_f >= 1 && p->n_fit >= 2 &&
           p->n_fit <= kMaxFit && p->sg_degree >= 1 && p->sg_degree <= 4 && p->sg_degree < p->n_fit &&
           p->k_a > 0.0 && p->a_targ >= 0.0 && p->table_nT >= 2 && p->table_meas >= 1 && p->table_burn >= 0 &&
           p->table_T_lo > 0.0 && p->table_T_hi > p->table_T_lo &&
           (p->tile_rows == 0 || shape_of(p->tile_rows) >= 0) &&
           p->sweeps_per_launch >= 0 && p->sweeps_per_launch <= 4096 && (p->spread == 0 || p->spread == 1) &&
           (p->fp64 == 0 || p->fp64 == 1) &&
           (p->table_side_cap == 0 || p->table_side_cap >= 2) && p->warm_min_states >= 0 && p->sweep_limit >= 0 &&
           (p->resume == 0 || p->resume == 1) && p->barrier_timeout_us >= 0;
}

bool valid_images(const mpr_image *imgs, int n)
{
    if (!imgs || n < 1) return false;
    for (int b = 0; b < n; ++b) {
        if (imgs[b].nx < 1 || imgs[b].ny < 1 || imgs[b].offset < 0) return false;
        if ((int64_t)imgs[b].nx * imgs[b].ny > (int64_t)1 << 31) return false;
        // the sweep kernels address a single-precision half-grid with 32-bit byte offsets
        if (half_grid_bytes(imgs[b].nx, imgs[b].ny) >= ((int64_t)1 << 32)) return false;
        if (imgs[b].id >= 0x80000000u) return false;
    }
    return true;
}

// Writes `hdr` (a run that cannot be resumed) over the header of a workspace
// at the end of its scope, unless d_hdr is null by then.
struct HeaderGuard {
    RunHeader *d_hdr;
    const RunHeader &hdr;
    hipStream_t stream;
    ~HeaderGuard()
    {
        if (!d_hdr) return;
        (void)hipMemcpyAsync(d_hdr, &hdr, sizeof hdr, hipMemcpyHostToDevice, stream);
        (void)hipStreamSynchronize(stream);
        (void)hipGetLastError();
    }
};

constexpr uint64_t kRunMagic = 0x4D50522D52554E31ull;  // "MPR-RUN1"
constexpr int64_t kRunHeaderBytes = 256;

int64_t sim_bytes(const mpr_image *imgs, int n, const mpr_params *p)
{
    int64_t b = kRunHeaderBytes;
    for (int i = 0; i < n; ++i) {
        const int64_t hg = round_up(half_grid_bytes(imgs[i].nx, imgs[i].ny, p->fp64 ? 8 : 4), 256);
        // angles (twice for single precision: the fused sweep's second buffer),
        // equilibrium sums, squared deviations
        b += (int64_t)p->R * 2 * hg * ((p->fp64 ? 1 : 2) + (p->K > 1 ? (p->spread ? 2 : 1) : 0));
    }
    const int64_t chains = (int64_t)n * p->R;
    b += round_up(chains * (int64_t)sizeof(ChainDesc), 256) + round_up(chains * (int64_t)sizeof(ChainState), 256);
    b += round_up(chains * 8, 256) + round_up((int64_t)n * sizeof(ImgDev), 256) + 4096;
    b += round_up(kNumStarts * (chains + 1) * 8, 256) + round_up(chains * 4 + 4, 256);
    for (int i = 0; i < n; ++i) b += redo_bytes(imgs[i].nx, imgs[i].ny, p->R);
    return b;
}

// FNV-1a over the images (size, offset, id), the parameters that shape a
// run's chains (all but sweep_limit, resume, tile_rows and
// sweeps_per_launch, which do not change its results) and the temperatures.
uint64_t run_key(const mpr_image *imgs, int n, const mpr_params *p, const double *T_hat)
{
    uint64_t h = 0xCBF29CE484222325ull;
    auto mix = [&h](const void *v, size_t len) {
        const unsigned char *b = (const unsigned char *)v;
        for (size_t i = 0; i < len; ++i) h = (h ^ b[i]) * 0x100000001B3ull;
    };
    mix(&n, sizeof n);
    for (int i = 0; i < n; ++i) {
        mix(&imgs[i].nx, 4);
        mix(&imgs[i].ny, 4);
        mix(&imgs[i].offset, 8);
        mix(&imgs[i].id, 4);
    }
    mpr_params q = *p;
    q.sweep_limit = 0;
    q.resume = 0;
    q.tile_rows = 0;
    q.sweeps_per_launch = 0;
    q.barrier_timeout_us = 0;
    mix(&q, sizeof q);
    mix(T_hat, sizeof(double) * (size_t)n);
    return h;
}

// Table chains run in double precision when q != 1/2 (the single-precision
// kernels are written for q = 1/2).
int table_angle_bytes(const mpr_params *p) { return p->q == 0.5 ? 4 : 8; }

// Grid on which the e(T, L) table of an image is built: its own, or each
// side capped at table_side_cap.
struct TableGrid {
    int32_t nx, ny;
};
TableGrid table_grid(const mpr_image &im, const mpr_params *p)
{
    const int32_t c = p->table_side_cap;
    return c > 0 ? TableGrid{std::min(im.nx, c), std::min(im.ny, c)} : TableGrid{im.nx, im.ny};
}

int64_t table_bytes(const mpr_image *imgs, int n, const mpr_params *p)
{
    int64_t best = 0;
    for (int i = 0; i < n; ++i) {
        const TableGrid t = table_grid(imgs[i], p);
        const int64_t hg = round_up(half_grid_bytes(t.nx, t.ny, table_angle_bytes(p)), 256);
        best = std::max(best, (int64_t)p->table_nT * 2 * hg);
    }
    const int64_t chains = p->table_nT;
    best += round_up(chains * (int64_t)sizeof(ChainDesc), 256) + round_up(chains * (int64_t)sizeof(ChainState), 256);
    best += round_up(chains * 8, 256) + round_up((int64_t)n * sizeof(ImgDev), 256) + 4096;
    best += round_up((int64_t)n * kMapBlocks * 16, 256);
    best += round_up(kNumStarts * (chains + 1) * 8, 256) + round_up(chains * 4 + 4, 256);
    int64_t rb = 0;
    for (int i = 0; i < n; ++i) {
        const TableGrid t = table_grid(imgs[i], p);
        rb = std::max(rb, redo_bytes(t.nx, t.ny, chains));
    }
    return best + rb;
}

// Derivative at the newest point of the degree-d least-squares polynomial
// through n equally spaced points, as weights on the values (oldest first):
// w = V (V^T V)^{-1} g with V_jk = s_j^k, s_j = j - (n-1)/2, g_k = k s_end^(k-1).
void sg_weights(int n, int degree, double *w)
{
    const int m = degree + 1;
    std::vector<double> A(m * m, 0.0), G(m, 0.0);
    const double c = 0.5 * (n - 1);
    for (int k = 0; k < m; ++k)
        for (int l = 0; l < m; ++l) {
            double s = 0.0;
            for (int j = 0; j < n; ++j) s += std::pow(j - c, k + l);
            A[k * m + l] = s;
        }
    const double send = (n - 1) - c;
    for (int k = 1; k < m; ++k) G[k] = k * std::pow(send, k - 1);
    // solve A x = G (A symmetric positive definite) by Gaussian elimination
    std::vector<double> M(A), x(G);
    for (int col = 0; col < m; ++col) {
        int piv = col;
        for (int r = col + 1; r < m; ++r)
            if (std::fabs(M[r * m + col]) > std::fabs(M[piv * m + col])) piv = r;
        if (piv != col) {
            for (int l = 0; l < m; ++l) std::swap(M[col * m + l], M[piv * m + l]);
            std::swap(x[col], x[piv]);
        }
        for (int r = col + 1; r < m; ++r) {
            const double f = M[r * m + col] / M[col * m + col];
            for (int l = col; l < m; ++l) M[r * m + l] -= f * M[col * m + l];
            x[r] -= f * x[col];
        }
    }
    for (int r = m - 1; r >= 0; --r) {
        double s = x[r];
        for (int l = r + 1; l < m; ++l) s -= M[r * m + l] * x[l];
        x[r] = s / M[r * m + r];
    }
    for (int j = 0; j < n; ++j) {
        double s = 0.0;
        for (int k = 0; k < m; ++k) s += std::pow(j - c, k) * x[k];
        w[j] = s;
    }
}

CtlParams make_ctl(const mpr_params *p)
{
    CtlParams cp;
    std::memset(&cp, 0, sizeof cp);
    cp.a_targ = p->a_targ;
    cp.k_a = p->k_a;
    cp.q = p->q;
    cp.n_f = p->n_f;
    cp.n_fit = p->n_fit;
    cp.i_max = p->i_max;
    cp.fixed_relax = p->fixed_relax;
    cp.eq_a_mode = p->eq_a_mode;
    cp.K = p->K;
    cp.burn = p->table_burn;
    cp.meas = p->table_meas;
    cp.e_unit = kEnergyUnit;
    cp.angle_bytes = 4;
    sg_weights(p->n_fit, p->sg_degree, cp.w);
    return cp;
}

SweepConsts make_sc(double q, uint64_t seed)
{
    SweepConsts sc;
    sc.q64 = q;
    sc.seed_lo = (uint32_t)seed;
    sc.seed_hi = (uint32_t)(seed >> 32);
    return sc;
}

int blocks_for(int64_t n, int cap) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + kBlock - 1) / kBlock, cap)); }


// A set of chains resident in the workspace.
struct ChainSet {
    std::vector<ChainDesc> desc;
    std::vector<ChainState> state;
    std::vector<int64_t> offset;  // image offset per chain (init)
    ChainDesc *d_desc = nullptr;
    ChainState *d_state = nullptr;
    int64_t *d_offset = nullptr;
    // the chains a sweep launch covers (those not done when the launch list
    // was last built): block prefix sums per shape and chain ids
    int64_t *d_start[kNumStarts] = {};
    int32_t *d_ids = nullptr;
    int n_active = 0;
    int64_t total_blocks[kNumShapes] = {};
    std::vector<int64_t> h_start;  // host copies (kept until their upload is done)
    std::vector<int32_t> h_ids;
    std::vector<char> upload;      // host copy of the descriptors' upload, unless it is staged in pinned memory
    Redo redo = {nullptr, nullptr};      // deferred double-precision updates
    int64_t redo_mask_bytes = 0, redo_bits_bytes = 0;
    bool redo_clean = false;             // both zeroed
    bool fp64 = false;                   // double-precision chains (no deferred redo)
    float *states_out = nullptr;         // recorded equilibrium states (nullable)
    int64_t states_n_total = 0;          // sites of the whole batch (stride of a state)
    int K = 0;
};

BlockMap block_map(const ChainSet &cs, int v) { return BlockMap{cs.d_start[start_of(v)], cs.d_ids, cs.n_active, 0}; }

template <int ROWS>
void launch_half_rows(hipStream_t st, const ChainSet &cs, int v, bool table, int colour, const SweepConsts &sc)
{
    const dim3 grid((unsigned)cs.total_blocks[v]);
    if (table)
        hipLaunchKernelGGL(table_half_sweep_kernel<ROWS>, grid, dim3(kBlock), 0, st, cs.d_desc, cs.d_state,
                           block_map(cs, v), colour, sc, cs.redo);
    else
        hipLaunchKernelGGL((half_sweep_kernel<false, ROWS>), grid, dim3(kBlock), 0, st, cs.d_desc, cs.d_state,
                           block_map(cs, v), colour, sc, 0, cs.redo, nullptr);
}

template <int CR>
void launch_half_compact(hipStream_t st, const ChainSet &cs, int v, int colour, const SweepConsts &sc)
{
    hipLaunchKernelGGL((half_sweep_compact_kernel<false, CR>), dim3((unsigned)cs.total_blocks[v]), dim3(kBlock), 0,
                       st, cs.d_desc, cs.d_state, block_map(cs, v), colour, sc, 0, cs.redo, nullptr);
}

// The deferred double-precision updates after a half-sweep in shape v.
template <bool DIAG>
void launch_redo(hipStream_t st, const ChainSet &cs, int v, int colour, const SweepConsts &sc, int or_only,
                 uint8_t *flags, const FusedControl *ctl = nullptr)
{
    FusedControl fc;
    if (ctl) fc = *ctl;
    else std::memset(&fc, 0, sizeof fc);
    // a wave per bitmap word, at most 16384 waves
    const int64_t nw = (cs.total_blocks[v] + 31) / 32;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((nw + 3) / 4, 4096));
    hipLaunchKernelGGL((redo_fp64_kernel<DIAG>), dim3(grid), dim3(kBlock), 0, st, cs.d_desc, cs.d_state,
                       block_map(cs, v), cs.total_blocks[v], kShapes[v].rows,
                       kShapes[v].compact ? 1 : 0, colour, sc, or_only, cs.redo, flags, fc);
}

template <bool DIAG, int ROWS>
void launch_half_fp64_rows(hipStream_t st, const ChainSet &cs, int v, int colour, const SweepConsts &sc, int or_only,
                           uint8_t *flags)
{
    hipLaunchKernelGGL((half_sweep_fp64_kernel<DIAG, ROWS>), dim3((unsigned)cs.total_blocks[v]), dim3(kBlock), 0, st,
                       cs.d_desc, cs.d_state, block_map(cs, v), colour, sc, or_only, flags);
}

template <bool DIAG, int CR>
void launch_half_fp64_compact(hipStream_t st, const ChainSet &cs, int v, int colour, const SweepConsts &sc,
                              int or_only, uint8_t *flags)
{
    hipLaunchKernelGGL((half_sweep_fp64_compact_kernel<DIAG, CR>), dim3((unsigned)cs.total_blocks[v]), dim3(kBlock),
                       0, st, cs.d_desc, cs.d_state, block_map(cs, v), colour, sc, or_only, flags);
}

// One half-sweep of double-precision chains in shape v.
template <bool DIAG>
void launch_half_fp64(hipStream_t st, const ChainSet &cs, int v, int colour, const SweepConsts &sc, int or_only,
                      uint8_t *flags)
{
    if (kShapes[v].compact) {
        switch (kShapes[v].rows) {
            case 2: launch_half_fp64_compact<DIAG, 2>(st, cs, v, colour, sc, or_only, flags); break;
            case 4: launch_half_fp64_compact<DIAG, 4>(st, cs, v, colour, sc, or_only, flags); break;
            default: launch_half_fp64_compact<DIAG, 8>(st, cs, v, colour, sc, or_only, flags); break;
        }
        return;
    }
    switch (kShapes[v].rows) {
        case 1: launch_half_fp64_rows<DIAG, 1>(st, cs, v, colour, sc, or_only, flags); break;
        case 2: launch_half_fp64_rows<DIAG, 2>(st, cs, v, colour, sc, or_only, flags); break;
        case 4: launch_half_fp64_rows<DIAG, 4>(st, cs, v, colour, sc, or_only, flags); break;
        default: launch_half_fp64_rows<DIAG, 8>(st, cs, v, colour, sc, or_only, flags); break;
    }
}

// One half-sweep of every chain in shape v (the e(T, L) runs use the plain
// shapes only); `ctl` (single precision only) makes the redo kernel run the
// per-sweep control as well.
void launch_half(hipStream_t st, const ChainSet &cs, int v, bool table, int colour, const SweepConsts &sc,
                 const FusedControl *ctl = nullptr)
{
    if (cs.fp64) {
        launch_half_fp64<false>(st, cs, v, colour, sc, 0, nullptr);
        return;
    }
    const Shape sh = kShapes[v];
    if (sh.compact && !table) {
        switch (sh.rows) {
            case 2: launch_half_compact<2>(st, cs, v, colour, sc); break;
            case 4: launch_half_compact<4>(st, cs, v, colour, sc); break;
            default: launch_half_compact<8>(st, cs, v, colour, sc); break;
        }
    } else {
        switch (sh.rows) {
            case 1: launch_half_rows<1>(st, cs, v, table, colour, sc); break;
            case 2: launch_half_rows<2>(st, cs, v, table, colour, sc); break;
            case 4: launch_half_rows<4>(st, cs, v, table, colour, sc); break;
            default: launch_half_rows<8>(st, cs, v, table, colour, sc); break;
        }
    }
    launch_redo<false>(st, cs, v, colour, sc, 0, nullptr, ctl);
}

// One fused sweep of every listed chain in shape v (mode 0), or one colour
// of it in place (mode 1, 2: diagnostics).
template <bool DIAG>
void launch_tile(hipStream_t st, const ChainSet &cs, int v, int mode, const SweepConsts &sc, int or_only,
                 uint8_t *flags, const FusedControl *ctl = nullptr)
{
    FusedControl fc;
    if (ctl) fc = *ctl;
    else std::memset(&fc, 0, sizeof fc);
    const dim3 grid((unsigned)cs.total_blocks[v]), blk(kBlock);
    switch (kShapes[v].rows) {
        case 16:
            hipLaunchKernelGGL((sweep_tile_kernel<DIAG, 16>), grid, blk, 0, st, cs.d_desc, cs.d_state,
                               block_map(cs, v), mode, sc, or_only, flags, fc);
            break;
        case 24:
            hipLaunchKernelGGL((sweep_tile_kernel<DIAG, 24>), grid, blk, 0, st, cs.d_desc, cs.d_state,
                               block_map(cs, v), mode, sc, or_only, flags, fc);
            break;
        case 48:
            hipLaunchKernelGGL((sweep_tile_kernel<DIAG, 48>), grid, blk, 0, st, cs.d_desc, cs.d_state,
                               block_map(cs, v), mode, sc, or_only, flags, fc);
            break;
        case 8:
            hipLaunchKernelGGL((sweep_tile_kernel<DIAG, 8>), grid, blk, 0, st, cs.d_desc, cs.d_state,
                               block_map(cs, v), mode, sc, or_only, flags, fc);
            break;
        case 12:
            hipLaunchKernelGGL((sweep_tile_kernel<DIAG, 12>), grid, blk, 0, st, cs.d_desc, cs.d_state,
                               block_map(cs, v), mode, sc, or_only, flags, fc);
            break;
        default:
            hipLaunchKernelGGL((sweep_tile_kernel<DIAG, 32>), grid, blk, 0, st, cs.d_desc, cs.d_state,
                               block_map(cs, v), mode, sc, or_only, flags, fc);
            break;
    }
}

template <typename RT, int TH>
const void *resident_kernel()
{
    static_assert((int64_t)kResMaxBlocks * res_halo_words<RT, TH>() * 8 <= (int64_t)kHaloBytes, "halo words");
    return reinterpret_cast<const void *>(&sweep_resident_kernel<RT, TH>);
}

// The resident kernel of a number of tile rows, null where there is none
// (tall tiles of doubles would leave no room for a second block on a CU).
const void *resident_kernel_of(int rows, bool fp64)
{
    switch (rows) {
        case 8: return fp64 ? resident_kernel<double, 8>() : resident_kernel<float, 8>();
        case 12: return fp64 ? resident_kernel<double, 12>() : resident_kernel<float, 12>();
        case 16: return fp64 ? resident_kernel<double, 16>() : resident_kernel<float, 16>();
        case 24: return fp64 ? resident_kernel<double, 24>() : resident_kernel<float, 24>();
        case 32: return fp64 ? resident_kernel<double, 32>() : resident_kernel<float, 32>();
        case 48: return fp64 ? nullptr : resident_kernel<float, 48>();
        case kResMaxRows: return fp64 ? nullptr : resident_kernel<float, kResMaxRows>();
        default: return nullptr;
    }
}

// Blocks of the resident sweep kernel that the device holds at once, 0
// without cooperative launches; cached on the context.
int64_t persist_capacity(mpr_ctx *ctx, int rows, bool fp64)
{
    const auto key = std::make_pair(rows, fp64 ? 8 : 4);
    auto it = ctx->persist_cap.find(key);
    if (it != ctx->persist_cap.end()) return it->second;
    int coop = 0, cus = 0, per_cu = 0;
    int64_t cap = 0;
    const void *f = resident_kernel_of(rows, fp64);
    if (f && hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, ctx->device) == hipSuccess && coop &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device) == hipSuccess &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, kResThreads, 0) == hipSuccess)
        cap = std::min<int64_t>((int64_t)per_cu * cus, kResMaxBlocks);
    (void)hipGetLastError();
    ctx->persist_cap[key] = cap;
    return cap;
}

// Up to rc.count fused sweeps of every listed chain in resident shape v, in
// one cooperative launch.
hipError_t launch_resident(mpr_ctx *ctx, hipStream_t st, const ChainSet &cs, int v, const SweepConsts &sc,
                           const CtlParams &cp, ResidentCtl rc, uint32_t start_ticks)
{
    if (ctx->halo_epoch == 0 || ctx->halo_epoch + 1 >= kResEpochs) {
        // no word may hold the tag of a later launch
        hipLaunchKernelGGL(clear_halo_kernel, dim3(512), dim3(kBlock), 0, st, rc.halo, (int64_t)kHaloBytes / 8);
        ctx->halo_epoch = 0;
    }
    rc.epoch = ++ctx->halo_epoch << kResSweepBits;
    hipLaunchKernelGGL(clear_resident_kernel, dim3(1), dim3(kBlock), 0, st, rc.gen, start_ticks, rc.sums,
                       3 * kResMaxBlocks);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const ChainDesc *descs = cs.d_desc;
    ChainState *states = cs.d_state;
    BlockMap bm = block_map(cs, v);
    SweepConsts scc = sc;
    CtlParams cpp = cp;
    void *args[] = {&descs, &states, &bm, &scc, &cpp, &rc};
    return hipLaunchCooperativeKernel(resident_kernel_of(kShapes[v].rows, cs.fp64), dim3((unsigned)cs.total_blocks[v]),
                                      dim3(kResThreads), args, 0, st);
}

// The launch list of a chain set from the chains in `active`: block prefix
// sums for every shape and the chain ids, in the set's host copies.
int list_active(mpr_ctx *ctx, ChainSet &cs, const std::vector<int32_t> &active)
{
    const int n = (int)cs.desc.size();
    const int na = (int)active.size();
    cs.h_start.assign((size_t)kNumStarts * (n + 1), 0);
    for (int k = 0; k < kNumShapes; ++k) {
        int64_t *sk = cs.h_start.data() + (size_t)start_of(k) * (n + 1);
        sk[0] = 0;
        for (int j = 0; j < na; ++j) sk[j + 1] = sk[j] + chain_blocks(cs.desc[active[j]], k);
        cs.total_blocks[k] = sk[na];
        if (sk[na] >= ((int64_t)1 << 31)) return fail(ctx, MPR_ERR_ARG, "batch too large for one launch");
    }
    cs.h_ids = active;
    cs.n_active = na;
    return MPR_OK;
}

// list_active, uploaded on `stream` and waited for, so that the host copies
// can be reused.
int set_active(mpr_ctx *ctx, ChainSet &cs, const std::vector<int32_t> &active, hipStream_t stream)
{
    if (int rc = list_active(ctx, cs, active)) return rc;
    HIP_TRY(ctx, hipMemcpyAsync(cs.d_start[0], cs.h_start.data(), cs.h_start.size() * 8, hipMemcpyHostToDevice,
                                stream));
    if (cs.n_active > 0)
        HIP_TRY(ctx, hipMemcpyAsync(cs.d_ids, cs.h_ids.data(), (size_t)cs.n_active * 4, hipMemcpyHostToDevice, stream));
    HIP_TRY(ctx, hipStreamSynchronize(stream));
    return MPR_OK;
}

// Zeroes the deferred-redo buffers of a chain set (the half-sweep shapes
// leave them zero).
int clear_redo(mpr_ctx *ctx, ChainSet &cs, hipStream_t stream)
{
    if (cs.redo_clean) return MPR_OK;
    HIP_TRY(ctx, hipMemsetAsync(cs.redo.mask, 0, (size_t)cs.redo_mask_bytes, stream));
    HIP_TRY(ctx, hipMemsetAsync(cs.redo.blocks, 0, (size_t)cs.redo_bits_bytes, stream));
    cs.redo_clean = true;
    return MPR_OK;
}

// Runs sweeps until every chain is done.  Returns 0 or an error code.
// A few direct sweeps per block shape come first (to tune it, unless fixed or
// cached), then groups of `spl` sweeps, those of the half-sweep shapes replayed
// as a captured graph (launched directly when `graphs` is false: instantiating
// a graph allocates), checking the done-counter after each group.  At most
// max_sweeps sweeps run; chains still running then are an error, or with
// `stop_ok` the result MPR_INCOMPLETE.
int run_chains(mpr_ctx *ctx, ChainSet &cs, const mpr_params *p, hipStream_t stream, int64_t max_sweeps,
               int poll_every, bool table, bool graphs = true, bool stop_ok = false)
{
    const int n = (int)cs.desc.size();
    unsigned int *d_done = reinterpret_cast<unsigned int *>((char *)ctx->scratch + kDoneOffset);
    unsigned int *d_ticket = reinterpret_cast<unsigned int *>((char *)ctx->scratch + kTicketOffset);
    unsigned long long *d_work = reinterpret_cast<unsigned long long *>((char *)ctx->scratch + kWorkOffset);
    unsigned int *d_gen = reinterpret_cast<unsigned int *>((char *)ctx->scratch + kGenOffset);
    unsigned int *d_abort = reinterpret_cast<unsigned int *>((char *)ctx->scratch + kAbortOffset);
    hipLaunchKernelGGL(clear_words_kernel, dim3(1), dim3(kBlock), 0, stream, d_done, d_abort, d_ticket, nullptr, 0);
    HIP_TRY(ctx, hipGetLastError());
    unsigned int already = 0;
    for (const auto &s : cs.state)
        if (s.phase == PH_DONE) ++already;
    if (already == (unsigned int)n) return MPR_OK;
    CtlParams cp = make_ctl(p);
    if (cs.fp64) {
        cp.e_unit = kEnergyUnit64;
        cp.angle_bytes = 8;
    }
    const SweepConsts sc = make_sc(p->q, p->seed);
    const int cblocks = (n + 63) / 64;
    hipStream_t st = stream;  // the context's own for shapes that are not resident

    // the control runs at the end of the colour-1 redo kernel unless
    // something must run between them (the state record) or there is no
    // redo kernel (double-precision chains)
    const bool fuse = !cs.fp64 && !cs.states_out;
    FusedControl fc;
    std::memset(&fc, 0, sizeof fc);
    fc.cp = cp;
    fc.ticket = d_ticket;
    fc.done_count = d_done;
    fc.work = d_work;
    fc.n_all = n;
    fc.on = 1;
    auto control = [&](int swap, int ctl) {
        hipLaunchKernelGGL(control_kernel, dim3(cblocks), dim3(64), 0, st, cs.d_desc, cs.d_state, n, cp, d_done,
                           d_work, swap, ctl);
    };
    // A sweep: the fused tile sweep, then control_kernel with the swap of
    // h and h2 (and the control, unless the states are recorded in between);
    // a fused sweep of at most kTileCtlMaxBlocks blocks does the swap and the
    // control in each chain's last block (unless states are recorded); or two
    // half-sweeps, the colour-1 redo kernel running the control unless the
    // states are recorded (or the chains are double precision).
    // The resident shapes: chain sets whose tiles the device holds at once.
    auto fits = [&](int v) {
        return kShapes[v].persist && cs.total_blocks[v] > 0 &&
               cs.total_blocks[v] <= persist_capacity(ctx, kShapes[v].rows, cs.fp64);
    };
    ResidentCtl rc0;
    std::memset(&rc0, 0, sizeof rc0);
    rc0.gen = d_gen;
    rc0.abort = d_abort;
    rc0.sums = reinterpret_cast<unsigned long long *>((char *)ctx->scratch + kSlotsOffset);
    rc0.halo = reinterpret_cast<unsigned long long *>((char *)ctx->scratch + kScratchBytes);
    rc0.done_count = d_done;
    rc0.work = d_work;
    rc0.states_out = cs.states_out;
    rc0.offsets = cs.d_offset;
    rc0.states_n_total = cs.states_n_total;
    rc0.K = cs.K;
    // The caller's bound on a block's wait holds where MPR_TILE_PERSIST can be
    // asked for: single-precision chains that record no states, in tiles of at
    // most 32 rows from the call's start.  Elsewhere resident sweeps stand in
    // for launches that wait for nothing: a launch that does not go within the
    // bound is called off, and no other bound below the default ends the call.
    const uint64_t own_wait = (uint64_t)p->barrier_timeout_us * 100u;
    bool tail = false;  // the last chains of a set, made resident on the way
    auto bounded = [&](int v) { return own_wait > 0 && fuse && !table && !tail && kShapes[v].rows <= 32; };
    bool called_off = false;  // a resident launch was: one launch per sweep from then on
    hipError_t perr = hipSuccess;
    auto sweeps = [&](int v, int count) {
        if (kShapes[v].persist) {
            rc0.wait_ticks = bounded(v) ? own_wait : std::max(own_wait, kPersistWaitTicks);
            rc0.count = count;
            const uint64_t start = own_wait > 0 ? std::min<uint64_t>(own_wait, UINT32_MAX) : kPersistStartTicks;
            perr = launch_resident(ctx, st, cs, v, sc, cp, rc0, (uint32_t)start);
            return;
        }
        for (int i = 0; i < count; ++i) {
            const bool fused = kShapes[v].fused;
            if (fused && fuse && cs.total_blocks[v] <= kTileCtlMaxBlocks) {
                launch_tile<false>(st, cs, v, 0, sc, 0, nullptr, &fc);  // swap and control in each chain's last block
            } else if (fused) {
                launch_tile<false>(st, cs, v, 0, sc, 0, nullptr);
                control(1, cs.states_out ? 0 : 1);
            } else {
                launch_half(st, cs, v, table, 0, sc);
                launch_half(st, cs, v, table, 1, sc, fuse ? &fc : nullptr);
            }
            if (cs.states_out && cs.n_active > 0)
                hipLaunchKernelGGL(record_states_kernel, dim3((unsigned)(cs.n_active * kRecordSegs)), dim3(kBlock), 0,
                                   st, cs.d_desc, cs.d_state, cs.d_offset, cs.d_ids, kRecordSegs, cs.K,
                                   cs.fp64 ? 1 : 0, cs.states_n_total, cs.states_out);
            if (fused ? cs.states_out != nullptr : !fuse) control(0, 1);
        }
    };
    int64_t done_sweeps = 0;
    bool finished = false;
    // Runs `count` sweeps directly or as graph `ge`, timed; then polls.
    auto block = [&](int v, int count, hipGraphExec_t ge, float *ms_out) -> int {
        const bool timed = ms_out || ctx->profile;
        if (!kShapes[v].fused && !cs.fp64)
            if (int rc = clear_redo(ctx, cs, st)) return rc;
        if (timed) HIP_TRY(ctx, hipEventRecord(ctx->ev_t0, st));
        if (ge) HIP_TRY(ctx, hipGraphLaunch(ge, st));
        else sweeps(v, count);
        if (perr != hipSuccess) return fail(ctx, MPR_ERR_HIP, "persistent sweep launch: %s", hipGetErrorString(perr));
        HIP_TRY(ctx, hipGetLastError());
        if (timed) HIP_TRY(ctx, hipEventRecord(ctx->ev_t1, st));
        // the done counter; after a resident launch the words up to the
        // abort word, in one copy (done counter, sweeps run, abort word)
        HIP_TRY(ctx, hipMemcpyAsync(ctx->done_host, d_done,
                                    kShapes[v].persist ? (size_t)(kAbortOffset + 4) : sizeof(unsigned int),
                                    hipMemcpyDeviceToHost, st));
        HIP_TRY(ctx, hipStreamSynchronize(st));
        if (kShapes[v].persist) {
            called_off = ctx->done_host[kGenOffset / 4 + kResGoes] == kResOff;
            if (ctx->done_host[kAbortOffset / 4] != 0u || (called_off && bounded(v)))
                return fail(ctx, MPR_ERR_HIP,
                            "resident sweeps: a block waited for another one longer than its bound (2 s, or "
                            "params.barrier_timeout_us)");
            // the launch stops early once every chain is done
            count = (int)ctx->done_host[kGenOffset / 4];
        }
        float ms = 0.0f;
        if (timed) HIP_TRY(ctx, hipEventElapsedTime(&ms, ctx->ev_t0, ctx->ev_t1));
        if (ms_out) *ms_out = ms;
        if (ctx->profile) {
            ctx->prof_ms += ms;
            ctx->prof_launches += (kShapes[v].fused ? 1 : 2) * (int64_t)count;
        }
        done_sweeps += count;
        finished = *ctx->done_host + already >= (unsigned int)n;
        return MPR_OK;
    };

    // block shape: fixed, resident, or else tuned on the first sweeps.  The one
    // launch per sweep shapes of table chains are the plain ones, those of
    // double-precision chains every unfused one.
    const int n_shapes = table ? kNumPlainShapes : (cs.fp64 ? kNumUnfusedShapes : kNumShapes);
    const int per_sweep = table || cs.fp64 ? kDefaultShape : shape_of(32 | MPR_TILE_FUSED);
    int v = p->tile_rows ? shape_of(p->tile_rows) : -1;
    if (v >= n_shapes) v = kDefaultShape;
    // a resident shape asked for whose tiles the device does not hold at once:
    // the smallest taller one it does, or else its rows, one launch per sweep
    if (v >= 0 && kShapes[v].persist && !fits(v)) {
        int t = v + 1;
        while (t < kNumShapes && !fits(t)) ++t;
        v = t < kNumShapes ? t : shape_of(kShapes[v].rows | MPR_TILE_FUSED);
    }
    int64_t sites = 0, gaps = 0;
    for (const auto &d : cs.desc) {
        sites += (int64_t)d.nx * d.ny;
        gaps += d.P;
    }
    // The resident shape of a chain set, or -1 if its tiles do not fit.
    // 1. The lowest tiles that leave a CU for each block, else the lowest that
    //    fit.  Low tiles spread a sweep over more waves, but a second block on
    //    a CU takes its share of the issue slots: us per sweep in relaxation /
    //    equilibrium, half gaps, 1024^2: 16 rows (512 blocks) 13.3 / 6.9, 32
    //    rows (256) 10.0 / 6.7, 64 rows (128) 12.6 / 10.6; 16 chains of 128^2:
    //    8 rows (256) 6.3 / 4.4, 16 rows (128) 6.8 / 5.1; 1500^2, 66%, whole
    //    fill: 48 rows (384) 959 us, 64 rows (288) 1064.
    // 2. At least 16 rows below an eighth of gaps: the waves of an 8-row block
    //    are left with nothing to do (fills of 4 chains of 256^2, 5% gaps: 8
    //    rows 308 us, 16 rows 292; 66%: 421 and 450).
    // 3. Not above 32 rows if lower tiles fit and most sweeps are equilibrium
    //    ones (100 states and more), which wait for no other block than the
    //    neighbours (1350^2 in clouds, 40%, K = 100: 32 rows, 473 blocks 2070
    //    us, 64 rows, 242 blocks 2414), or if a chain is 3 to 16 tiles of 32
    //    rows: its blocks wait for few others, and chains that end leave their
    //    CU to the second block (128 chains of 128^2, 66%: 32 rows 1016 us, 64
    //    rows 1356; 24 of 256^2: 804 and 926; but 8 of 512^2, 64 blocks each:
    //    990 and 916).
    // Over 428 fills (64^2 to 1900 x 700, 1 to 256 chains, 5 to 90% gaps, random
    // and clouds, both precisions) the shape taken is within 5% of the best in
    // nine of ten.  One launch per sweep takes 1.2 to 3 times as long.
    auto resident_shape = [&]() {
        int best = -1, low = -1, rows32 = -1;
        for (int k = 0; k < kNumShapes; ++k) {
            if (!fits(k) || (kShapes[k].rows < 16 && 8 * gaps < sites)) continue;
            if (low < 0) low = k;
            if (kShapes[k].rows == 32) rows32 = k;
            if (best < 0 || (cs.total_blocks[best] > kResMaxBlocks / 2 && cs.total_blocks[k] <= kResMaxBlocks / 2))
                best = k;
        }
        if (rows32 >= 0 && kShapes[best].rows > 32) {
            const int64_t blocks = cs.total_blocks[rows32], na = cs.n_active;
            if (cs.K >= 100) best = low;
            else if (blocks >= 3 * na && blocks <= 16 * na) best = rows32;
        }
        return best;
    };
    if (v < 0) v = resident_shape();
    // The resident shapes run on the caller's stream, the others on the
    // context's own, ordered after and before the caller's with two events (15
    // to 40 us of a call): half-sweeps are captured into graphs (the caller's
    // may be the default stream, which cannot be captured, and other threads
    // may use it), and calls of several threads on the default stream overlap.
    if (v < 0 || !kShapes[v].persist) {
        st = ctx->gstream;
        HIP_TRY(ctx, hipEventRecord(ctx->ev_in, stream));
        HIP_TRY(ctx, hipStreamWaitEvent(st, ctx->ev_in, 0));
    }
    float sweep_ms = -1.0f;
    if (v < 0) {
        int maxnx = 0, maxny = 0;
        for (const auto &d : cs.desc) {
            maxnx = std::max(maxnx, d.nx);
            maxny = std::max(maxny, d.ny);
        }
        const int kind = (table ? 1 : 0) | (cs.fp64 ? 2 : 0) | (cs.states_out ? 4 : 0) | (cs.desc[0].acc[0] ? 8 : 0) |
                         (cs.desc[0].m2[0] ? 16 : 0);
        mpr_ctx::Tuned &tn = ctx->tuned_rows[std::make_tuple(kind, n, maxnx, maxny, cs.total_blocks[kSmallTileShape],
                                                             (int)(8 * gaps / sites))];
        const int ts = std::max(1, std::min(poll_every, 3));
        for (; tn.next < n_shapes && !finished && done_sweeps + ts <= max_sweeps; ++tn.next) {
            const int k = tn.next;
            if (kShapes[k].persist) continue;
            float ms = 0.0f;
            int rc = block(k, ts, nullptr, &ms);
            if (rc) return rc;
            ms /= (float)ts;
            if (tn.best < 0 || ms < tn.ms) {
                tn.ms = ms;
                tn.best = k;
            }
        }
        v = kDefaultShape;
        if (tn.best >= 0) {
            v = tn.best;
            sweep_ms = tn.ms;
        }
    }
    if (!table) ctx->last_tile = tile_code(kShapes[v]);
    // sweeps per graph: at least about a millisecond of work per done-check
    int spl = p->sweeps_per_launch > 0 ? p->sweeps_per_launch : poll_every;
    if (p->sweeps_per_launch <= 0 && sweep_ms > 0.0f && (float)spl * sweep_ms < 1.0f)
        spl = std::min(64, poll_every * (int)std::ceil(1.0f / ((float)poll_every * sweep_ms)));
    // a persistent launch ends by itself when every chain is done: a group
    // of 256 sweeps covers a whole small fill in one launch and one poll
    if (p->sweeps_per_launch <= 0 && kShapes[v].persist) spl = 256;
    // the captured sweep group, released on every return path
    struct Captured {
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
        void release()
        {
            if (exec) (void)hipGraphExecDestroy(exec);
            if (graph) (void)hipGraphDestroy(graph);
            exec = nullptr;
            graph = nullptr;
        }
        ~Captured() { release(); }
    } cap;
    hipGraphExec_t &ge = cap.exec;
    auto capture = [&]() {
        cap.release();
        // (a resident launch runs a whole group itself; a fused sweep is one or
        // two launches of 20 us and more, which the host keeps ahead of, and
        // capturing its graph anew whenever the list changes took 60 to 190 us)
        if (graphs && !kShapes[v].fused && st == ctx->gstream &&
            hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal) == hipSuccess) {
            sweeps(v, spl);
            if (hipStreamEndCapture(st, &cap.graph) != hipSuccess ||
                hipGraphInstantiate(&cap.exec, cap.graph, nullptr, nullptr, 0) != hipSuccess)
                cap.exec = nullptr;
        }
        (void)hipGetLastError();
    };
    if (!finished) capture();
    // Chains stop at different sweeps.  When at least an eighth of the
    // listed chains have finished, the launch list is rebuilt from the
    // chains still running if that drops a fifth or more of the blocks a
    // launch covers (the blocks of finished chains return at once, but
    // still have to be dispatched).
    unsigned int done_listed = already;
    std::vector<uint8_t> done_flag(n);
    uint8_t *d_flags = (uint8_t *)ctx->scratch + kVarOffset;
    const bool can_shrink = (int64_t)n <= (int64_t)kScratchBytes - kVarOffset;
    int rc = MPR_OK;
    while (!finished && done_sweeps < max_sweeps) {
        // the last group may be shorter: exactly max_sweeps sweeps run
        const int cnt = (int)std::min<int64_t>(spl, max_sweeps - done_sweeps);
        rc = block(v, cnt, cnt == spl ? ge : nullptr, nullptr);
        if (rc) break;
        if (called_off && kShapes[v].persist) {
            v = per_sweep;
            if (!table) ctx->last_tile = tile_code(kShapes[v]);
            if (p->sweeps_per_launch <= 0) spl = poll_every;
            capture();
            continue;
        }
        const unsigned int done_now = *ctx->done_host + already;
        if (finished || !can_shrink || done_now - done_listed < std::max(1u, (unsigned int)cs.n_active / 8u))
            continue;
        done_listed = done_now;
        hipLaunchKernelGGL(done_flags_kernel, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, st, cs.d_state, n,
                           d_flags);
        HIP_TRY(ctx, hipMemcpyAsync(done_flag.data(), d_flags, (size_t)n, hipMemcpyDeviceToHost, st));
        HIP_TRY(ctx, hipStreamSynchronize(st));
        std::vector<int32_t> active;
        int64_t blocks = 0;
        for (int c = 0; c < n; ++c)
            if (!done_flag[c]) {
                active.push_back(c);
                blocks += chain_blocks(cs.desc[c], v);
            }
        if (active.empty() || 5 * blocks > 4 * cs.total_blocks[v]) continue;
        rc = set_active(ctx, cs, active, st);
        if (rc) break;
        if (!p->tile_rows && !kShapes[v].persist && !called_off) {
            // the last chains of a set finish in one resident launch once
            // they fit
            const int best = resident_shape();
            if (best >= 0) {
                v = best;
                tail = true;
                if (p->sweeps_per_launch <= 0) spl = 256;
            }
        }
        capture();
    }
    cap.release();
    if (rc) return rc;
    if (st != stream) {
        HIP_TRY(ctx, hipEventRecord(ctx->ev_out, st));
        HIP_TRY(ctx, hipStreamWaitEvent(stream, ctx->ev_out, 0));
    }
    if (!finished)
        return stop_ok ? MPR_INCOMPLETE
                       : fail(ctx, MPR_ERR_HIP, "chains did not finish within %lld sweeps", (long long)max_sweeps);
    return MPR_OK;
}

ChainState fresh_state(double T, int phase)
{
    ChainState s;
    std::memset(&s, 0, sizeof s);
    s.phase = phase;
    s.sweep = 0;
    s.T = T;
    s.a_cur = 1.0;
    s.a_relax = 1.0;
    s.k = -1.0;
    s.inv_k = 1.0f;
    s.inv_km1 = 0.0f;
    s.inv_k_d = 1.0;
    s.inv_km1_d = 0.0;
    return s;
}

// Carves descriptors, states, launch list and deferred-redo buffers (sized for
// every chain) of a chain set from the workspace and uploads them, in one copy:
// they lie one after the other.  The launch list holds the chains that are not
// done.  With `resume` the states are read back from the workspace first (the
// run it holds), and each chain whose fused sweeps left h and h2 exchanged gets
// them exchanged in its descriptor too.
int upload_chains(mpr_ctx *ctx, ChainSet &cs, Carver &cv, hipStream_t stream, double q, bool resume = false)
{
    const int n = (int)cs.desc.size();
    cs.d_desc = (ChainDesc *)cv.take(n * (int64_t)sizeof(ChainDesc));
    cs.d_state = (ChainState *)cv.take(n * (int64_t)sizeof(ChainState));
    cs.d_offset = (int64_t *)cv.take(n * 8);
    int64_t *d = (int64_t *)cv.take((int64_t)kNumStarts * (n + 1) * 8);
    cs.d_ids = (int32_t *)cv.take((int64_t)n * 4 + 4);
    if (!cs.d_desc || !cs.d_state || !cs.d_offset || !d || !cs.d_ids)
        return fail(ctx, MPR_ERR_WORKSPACE, "workspace too small");
    for (int k = 0; k < kNumStarts; ++k) cs.d_start[k] = d + (size_t)k * (n + 1);
    int64_t words = 0, blocks = 0;
    for (int k = 0; k < kNumShapes; ++k) {
        int64_t b = 0;
        for (int c = 0; c < n; ++c) b += chain_blocks(cs.desc[c], k);
        words = std::max(words, b * redo_words(k));
        blocks = std::max(blocks, b);
    }
    cs.redo_mask_bytes = words * 4;
    cs.redo_bits_bytes = (blocks + 31) / 32 * 4;
    cs.redo.mask = (uint32_t *)cv.take(cs.redo_mask_bytes);
    cs.redo.blocks = (uint32_t *)cv.take(cs.redo_bits_bytes);
    cs.redo_clean = false;
    if (!cs.redo.mask || !cs.redo.blocks) return fail(ctx, MPR_ERR_WORKSPACE, "workspace too small");
    if (resume) {
        HIP_TRY(ctx, hipMemcpyAsync(cs.state.data(), cs.d_state, n * sizeof(ChainState), hipMemcpyDeviceToHost,
                                    stream));
        HIP_TRY(ctx, hipStreamSynchronize(stream));
        for (int c = 0; c < n; ++c)
            if (cs.state[c].swapped) {
                std::swap(cs.desc[c].h[0], cs.desc[c].h2[0]);
                std::swap(cs.desc[c].h[1], cs.desc[c].h2[1]);
            }
    } else {
        for (auto &s : cs.state) {
            s.inv_T = (float)(1.0 / s.T);
            s.dscale = (float)(kTwoPi * q / s.a_cur);
        }
    }
    std::vector<int32_t> active;
    for (int c = 0; c < n; ++c)
        if (cs.state[c].phase != PH_DONE) active.push_back(c);
    int rc = list_active(ctx, cs, active);
    if (rc) return rc;
    char *const base = (char *)cs.d_desc;
    const int64_t bytes = (char *)(cs.d_ids + n + 1) - base;
    char *h = stage_for(ctx, bytes, cs.upload);
    std::memset(h, 0, (size_t)bytes);
    std::memcpy(h, cs.desc.data(), n * sizeof(ChainDesc));
    std::memcpy(h + ((char *)cs.d_state - base), cs.state.data(), n * sizeof(ChainState));
    std::memcpy(h + ((char *)cs.d_offset - base), cs.offset.data(), (size_t)n * 8);
    std::memcpy(h + ((char *)d - base), cs.h_start.data(), cs.h_start.size() * 8);
    std::memcpy(h + ((char *)cs.d_ids - base), cs.h_ids.data(), cs.h_ids.size() * 4);
    HIP_TRY(ctx, hipMemcpyAsync(base, h, (size_t)bytes, hipMemcpyHostToDevice, stream));
    return MPR_OK;
}

// Allocates both half-grids (and accumulators) of a chain of `eb`-byte
// angles from the workspace.
bool carve_chain(Carver &cv, ChainDesc &d, int nx, int ny, bool with_acc, bool with_m2 = false, int eb = 4,
                 bool with_h2 = false)
{
    const int64_t hg = half_grid_bytes(nx, ny, eb);
    d.nx = nx;
    d.ny = ny;
    d.S = half_stride(nx);
    for (int c = 0; c < 2; ++c) {
        d.h[c] = (float *)cv.take(hg);
        d.h2[c] = with_h2 ? (float *)cv.take(hg) : nullptr;
        d.acc[c] = with_acc ? (float *)cv.take(hg) : nullptr;
        d.m2[c] = with_acc && with_m2 ? (float *)cv.take(hg) : nullptr;
        if (!d.h[c] || (with_h2 && !d.h2[c]) || (with_acc && !d.acc[c]) || (with_acc && with_m2 && !d.m2[c]))
            return false;
    }
    return true;
}

// Starting angles of every chain of a set (table: pi everywhere), and the
// run's header, if there is one.
void launch_init(hipStream_t stream, const ChainSet &cs, const float *phi, const uint8_t *sampled,
                 const float *phi_init, uint64_t seed, int table, const RunHeader &hdr = RunHeader{},
                 RunHeader *d_hdr = nullptr)
{
    int64_t groups = 1;
    for (const auto &d : cs.desc) groups = std::max(groups, (int64_t)d.ny * d.S / 2);
    const dim3 grid(blocks_for(groups, 2048), (unsigned)cs.desc.size());
    if (cs.fp64)
        hipLaunchKernelGGL(init_chains_kernel<double>, grid, dim3(kBlock), 0, stream, cs.d_desc, cs.d_offset, phi,
                           sampled, phi_init, (uint32_t)seed, (uint32_t)(seed >> 32), table, hdr, d_hdr);
    else
        hipLaunchKernelGGL(init_chains_kernel<float>, grid, dim3(kBlock), 0, stream, cs.d_desc, cs.d_offset, phi,
                           sampled, phi_init, (uint32_t)seed, (uint32_t)(seed >> 32), table, hdr, d_hdr);
}

// Monotone (pool-adjacent-violators) fit of y, then log T interpolated
// linearly in y; y = log(1 + e).
double invert_table(const std::vector<double> &Tg, const std::vector<double> &ope, double e_s, int *clamped)
{
    const int n = (int)Tg.size();
    std::vector<double> val, wt;
    std::vector<int> len;
    for (int k = 0; k < n; ++k) {
        val.push_back(std::log(std::max(ope[k], 1e-300)));
        wt.push_back(1.0);
        len.push_back(1);
        while (val.size() > 1 && val[val.size() - 2] > val.back()) {
            const double w2 = wt[wt.size() - 2] + wt.back();
            const double v2 = (wt[wt.size() - 2] * val[val.size() - 2] + wt.back() * val.back()) / w2;
            const int l2 = len[len.size() - 2] + len.back();
            val.pop_back();
            wt.pop_back();
            len.pop_back();
            val.back() = v2;
            wt.back() = w2;
            len.back() = l2;
        }
    }
    std::vector<double> y;
    for (size_t b = 0; b < val.size(); ++b)
        for (int j = 0; j < len[b]; ++j) y.push_back(val[b]);
    const double ys = std::log(std::max(1.0 + e_s, 1e-300));
    *clamped = 0;
    if (ys <= y[0]) {
        *clamped = 1;
        return Tg[0];
    }
    if (ys >= y[n - 1]) {
        *clamped = 1;
        return Tg[n - 1];
    }
    int k = 0;
    while (!(y[k + 1] >= ys && y[k + 1] > y[k])) ++k;
    const double x0 = std::log(Tg[k]), x1 = std::log(Tg[k + 1]);
    return std::exp(x0 + (ys - y[k]) * (x1 - x0) / (y[k + 1] - y[k]));
}

// Device address of static_workspace on `device` (the current device),
// looked up once per device and kept for the process.
std::mutex g_static_ws_mu;
void *g_static_ws_addr[kMaxDevices] = {};

hipError_t static_ws_addr(int device, void **out)
{
    *out = nullptr;
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_static_ws_mu);
    if (!g_static_ws_addr[device]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(static_workspace));
        if (e != hipSuccess) return e;
        g_static_ws_addr[device] = ptr;
    }
    *out = g_static_ws_addr[device];
    return hipSuccess;
}

std::vector<double> temperature_grid(const mpr_params *p)
{
    std::vector<double> Tg(p->table_nT);
    for (int k = 0; k < p->table_nT; ++k)
        Tg[k] = std::exp(std::log(p->table_T_lo) +
                         (std::log(p->table_T_hi) - std::log(p->table_T_lo)) * (double)k / (double)(p->table_nT - 1));
    return Tg;
}

}  // namespace

// ================================================================== C ABI

extern "C" {

int32_t mpr_create(mpr_ctx **out, int32_t device)
{
    if (!out) return MPR_ERR_ARG;
    *out = nullptr;
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || device < 0 || device >= count) return MPR_ERR_HIP;
    if (hipSetDevice(device) != hipSuccess) return MPR_ERR_HIP;
    mpr_ctx *ctx = new mpr_ctx();
    ctx->device = device;
    // without it only mpr_simulate_noalloc is unavailable (it reports so)
    if (static_ws_addr(device, &ctx->static_ws) != hipSuccess) {
        ctx->static_ws = nullptr;
        (void)hipGetLastError();
    }
    if (hipMalloc(&ctx->scratch, kScratchBytes + kHaloBytes) != hipSuccess ||
        hipHostMalloc((void **)&ctx->done_host, kHostStageBytes, hipHostMallocDefault) != hipSuccess ||
        hipStreamCreateWithFlags(&ctx->gstream, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&ctx->ev_in, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&ctx->ev_out, hipEventDisableTiming) != hipSuccess ||
        hipEventCreate(&ctx->ev_t0) != hipSuccess || hipEventCreate(&ctx->ev_t1) != hipSuccess) {
        mpr_destroy(ctx);
        return MPR_ERR_HIP;
    }
    *out = ctx;
    return MPR_OK;
}

void mpr_destroy(mpr_ctx *ctx)
{
    if (!ctx) return;
    (void)hipSetDevice(ctx->device);
    if (ctx->gstream) (void)hipStreamSynchronize(ctx->gstream);
    for (hipEvent_t ev : {ctx->ev_in, ctx->ev_out, ctx->ev_t0, ctx->ev_t1})
        if (ev) (void)hipEventDestroy(ev);
    if (ctx->gstream) (void)hipStreamDestroy(ctx->gstream);
    if (ctx->scratch) (void)hipFree(ctx->scratch);
    if (ctx->done_host) (void)hipHostFree(ctx->done_host);
    delete ctx;
}

const char *mpr_last_error(const mpr_ctx *ctx) { return ctx ? ctx->err.c_str() : "null context"; }

void mpr_default_params(mpr_params *p)
{
    if (!p) return;
    std::memset(p, 0, sizeof *p);
    p->q = 0.5;
    p->R = 1;
    p->K = 100;
    p->n_f = 5;
    p->n_fit = 20;
    p->sg_degree = 1;
    p->i_max = 20000;
    p->a_targ = 0.3;
    p->k_a = 3.0;
    p->fixed_relax = -1;
    p->eq_a_mode = 0;
    p->table_nT = 32;
    p->table_burn = 200;
    p->table_meas = 400;
    p->table_T_lo = 1e-5;
    p->table_T_hi = 10.0;
    p->seed = 3000;
    p->tile_rows = 0;
    p->sweeps_per_launch = 0;
    p->spread = 0;
    p->fp64 = 0;
    p->table_side_cap = 0;
    p->warm_min_states = kWarmMinStates;
}

int64_t mpr_workspace_size(const mpr_image *imgs, int32_t n, const mpr_params *p)
{
    if (!valid_images(imgs, n) || !valid_params(p)) return -1;
    return std::max(sim_bytes(imgs, n, p), table_bytes(imgs, n, p));
}

int32_t mpr_map_to_angles(mpr_ctx *ctx, const mpr_image *imgs, int32_t n, const float *z, const uint8_t *sampled,
                          float *phi, double *zmin_zmax, void *stream_)
{
    if (!ctx) return MPR_ERR_ARG;
    if (!valid_images(imgs, n) || !z || !sampled || !phi || !zmin_zmax)
        return fail(ctx, MPR_ERR_ARG, "map_to_angles: invalid argument");
    if (int rc = mpr_check_device(ctx, "map_to_angles", {{"z", z}, {"sampled", sampled}, {"phi", phi}})) return rc;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    hipStream_t stream = (hipStream_t)stream_;
    const int chunk = (int)((kScratchBytes - kVarOffset - 4096) / (kMapBlocks * 24 + 64));
    for (int b0 = 0; b0 < n; b0 += chunk) {
        const int nb = std::min(chunk, n - b0);
        char *sp = (char *)ctx->scratch + kVarOffset;
        ImgDev *d_img = (ImgDev *)sp;
        float *pmin = (float *)(sp + round_up((int64_t)nb * sizeof(ImgDev), 256));
        float *pmax = pmin + (int64_t)nb * kMapBlocks;
        unsigned long long *pcnt = (unsigned long long *)(pmax + (int64_t)nb * kMapBlocks);
        unsigned int *pbad = (unsigned int *)(pcnt + (int64_t)nb * kMapBlocks);
        double *d_zmm = (double *)(pbad + (int64_t)nb * kMapBlocks + 64);
        d_zmm = (double *)round_up((int64_t)d_zmm, 256);
        std::vector<ImgDev> hi;
        ImgArgs img;
        RangeArgs range;
        std::memset(&range, 0, sizeof range);
        if (int rc = image_args(ctx, stream, imgs + b0, nb, hi, d_img, img)) return rc;
        int mb = 1;  // partial blocks per image: the largest image's count (min, max and counts are exact)
        int64_t maxn = 0;
        for (int b = 0; b < nb; ++b) {
            mb = std::max(mb, minmax_blocks((int64_t)hi[b].nx * hi[b].ny));
            maxn = std::max(maxn, (int64_t)hi[b].nx * hi[b].ny);
        }
        hipLaunchKernelGGL(map_minmax_kernel, dim3(mb, nb), dim3(kBlock), 0, stream, img, z, sampled, pmin,
                           pmax, pcnt, pbad);
        HIP_TRY(ctx, hipGetLastError());
        if (n == 1) {
            // one image: its range goes from one kernel to the next on the
            // device, and one wait ends the call
            double *found = (double *)((char *)ctx->done_host + kHostWordsBytes);
            // (four sites a thread: every block reduces the partials first,
            // 10.6 us at 1024^2 with one site a thread, 7.7 with four)
            hipLaunchKernelGGL(map_apply_kernel, dim3(blocks_for((maxn + 3) / 4, 4096)), dim3(kBlock), 0, stream, img, range, mb,
                               pmin, pmax, pcnt, pbad, found, z, sampled, phi);
            HIP_TRY(ctx, hipGetLastError());
            HIP_TRY(ctx, hipStreamSynchronize(stream));
            if (found[3] != 0.0) return fail(ctx, MPR_ERR_ARG, "image 0: non-finite sampled value");
            if (found[2] < 2.0 || !(found[1] > found[0]))
                return fail(ctx, MPR_ERR_DEGENERATE, "image 0: fewer than 2 samples or z_max == z_min");
            zmin_zmax[0] = found[0];
            zmin_zmax[1] = found[1];
            return MPR_OK;
        }
        std::vector<float> hmin(nb * mb), hmax(nb * mb);
        std::vector<unsigned long long> hcnt(nb * mb);
        std::vector<unsigned int> hbad(nb * mb);
        // the four partial arrays lie one after the other: one copy
        {
            const char *src = (const char *)pmin;
            const int64_t span = (const char *)(pbad + (int64_t)nb * mb) - src;
            std::vector<char> big;
            char *h = stage_for(ctx, span, big);
            HIP_TRY(ctx, hipMemcpyAsync(h, src, (size_t)span, hipMemcpyDeviceToHost, stream));
            HIP_TRY(ctx, hipStreamSynchronize(stream));
            std::memcpy(hmin.data(), h + ((const char *)pmin - src), hmin.size() * 4);
            std::memcpy(hmax.data(), h + ((const char *)pmax - src), hmax.size() * 4);
            std::memcpy(hcnt.data(), h + ((const char *)pcnt - src), hcnt.size() * 8);
            std::memcpy(hbad.data(), h + ((const char *)pbad - src), hbad.size() * 4);
        }
        std::vector<double> zmm(2 * nb);
        for (int b = 0; b < nb; ++b) {
            float lo = INFINITY, hi2 = -INFINITY;
            unsigned long long cnt = 0;
            unsigned int bad = 0;
            for (int k = 0; k < mb; ++k) {
                lo = std::min(lo, hmin[b * mb + k]);
                hi2 = std::max(hi2, hmax[b * mb + k]);
                cnt += hcnt[b * mb + k];
                bad |= hbad[b * mb + k];
            }
            if (bad) return fail(ctx, MPR_ERR_ARG, "image %d: non-finite sampled value", b0 + b);
            if (cnt < 2 || !(hi2 > lo))
                return fail(ctx, MPR_ERR_DEGENERATE, "image %d: fewer than 2 samples or z_max == z_min", b0 + b);
            zmm[2 * b] = lo;
            zmm[2 * b + 1] = hi2;
            zmin_zmax[2 * (b0 + b)] = lo;
            zmin_zmax[2 * (b0 + b) + 1] = hi2;
        }
        if (int rc = range_args(ctx, stream, zmm.data(), nb, d_zmm, range)) return rc;
        hipLaunchKernelGGL(map_apply_kernel, dim3(blocks_for(maxn, 4096), nb), dim3(kBlock), 0, stream, img, range, 0,
                           nullptr, nullptr, nullptr, nullptr, nullptr, z, sampled, phi);
        HIP_TRY(ctx, hipGetLastError());
        HIP_TRY(ctx, hipStreamSynchronize(stream));
    }
    return MPR_OK;
}

int32_t mpr_estimate_temperature(mpr_ctx *ctx, const mpr_image *imgs, int32_t n, const float *phi,
                                 const uint8_t *sampled, const mpr_params *p, void *ws, int64_t ws_bytes,
                                 double *e_s, double *T_hat, int32_t *t_clamped, void *stream_)
{
    if (!ctx) return MPR_ERR_ARG;
    if (!valid_images(imgs, n) || !valid_params(p) || !phi || !sampled || !e_s || !T_hat)
        return fail(ctx, MPR_ERR_ARG, "estimate_temperature: invalid argument");
    if (!ws || ws_bytes < table_bytes(imgs, n, p)) return fail(ctx, MPR_ERR_WORKSPACE, "workspace too small");
    if (int rc = mpr_check_device(ctx, "estimate_temperature", {{"phi", phi}, {"sampled", sampled}, {"workspace", ws}}))
        return rc;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    hipStream_t stream = (hipStream_t)stream_;
    // e_s per image (equation mpr-sse)
    {
        Carver cv{(char *)ws, ws_bytes};
        ImgDev *d_img = (ImgDev *)cv.take(n * (int64_t)sizeof(ImgDev));
        double *psum = (double *)cv.take((int64_t)n * kMapBlocks * 8);
        unsigned long long *pcnt = (unsigned long long *)cv.take((int64_t)n * kMapBlocks * 8);
        if (!d_img || !psum || !pcnt) return fail(ctx, MPR_ERR_WORKSPACE, "workspace too small");
        std::vector<ImgDev> hi;
        ImgArgs img;
        if (int rc = image_args(ctx, stream, imgs, n, hi, d_img, img)) return rc;
        int mb = 1;  // the grid covers the largest image; each image uses image_blocks of its own size
        for (int b = 0; b < n; ++b) mb = std::max(mb, image_blocks((int64_t)hi[b].nx * hi[b].ny));
        // the partial sums and counts straight into pinned host memory where
        // they fit, else through the workspace and one copy
        const int64_t parts = (int64_t)n * mb;
        const bool direct = parts * 16 <= kHostStageBytes - kHostWordsBytes;
        std::vector<char> big;
        char *h = stage_for(ctx, direct ? parts * 16 : (const char *)(pcnt + parts) - (const char *)psum, big);
        double *os = direct ? (double *)h : psum;
        unsigned long long *oc = direct ? (unsigned long long *)(h + parts * 8) : pcnt;
        hipLaunchKernelGGL(sample_energy_kernel, dim3(mb, n), dim3(kEsThreads), 0, stream, img, phi, sampled, p->q, os, oc);
        HIP_TRY(ctx, hipGetLastError());
        if (!direct)
            HIP_TRY(ctx, hipMemcpyAsync(h, psum, (size_t)((const char *)(pcnt + parts) - (const char *)psum),
                                        hipMemcpyDeviceToHost, stream));
        HIP_TRY(ctx, hipStreamSynchronize(stream));
        const double *hs = (const double *)h;
        const unsigned long long *hc = (const unsigned long long *)(h + ((const char *)oc - (const char *)os));
        for (int b = 0; b < n; ++b) {
            double s = 0.0;
            unsigned long long c = 0;
            const int nbk = image_blocks((int64_t)hi[b].nx * hi[b].ny);
            for (int k = 0; k < nbk; ++k) {
                s += hs[(size_t)b * mb + k];
                c += hc[(size_t)b * mb + k];
            }
            if (c == 0) return fail(ctx, MPR_ERR_DEGENERATE, "image %d: no sample-sample pair", b);
            e_s[b] = s / (double)c;
        }
    }
    // e(T, L) tables per table grid size (equation ene), cached.  The
    // missing ones are built together: the table chains of as many grid
    // sizes as the workspace holds run as one ragged chain set (a table does
    // not depend on the chains run beside it: its random numbers are keyed by
    // temperature index and site).
    const std::vector<double> Tg = temperature_grid(p);
    std::vector<TableGrid> tg(n);
    for (int b = 0; b < n; ++b) tg[b] = table_grid(imgs[b], p);
    auto key_of = [&](int b) {
        return std::make_tuple(tg[b].nx, tg[b].ny, p->q, p->table_nT, p->table_T_lo, p->table_T_hi, p->table_burn,
                               p->table_meas, p->a_targ, p->k_a, p->seed);
    };
    std::vector<int> missing;  // first image of each table grid size without a table
    for (int b = 0; b < n; ++b) {
        if (ctx->tables.count(key_of(b))) continue;
        if ((int64_t)tg[b].nx * tg[b].ny < 2) return fail(ctx, MPR_ERR_DEGENERATE, "image %d: one site", b);
        bool dup = false;
        for (int m : missing) dup = dup || (tg[m].nx == tg[b].nx && tg[m].ny == tg[b].ny);
        if (!dup) missing.push_back(b);
    }
    const int nT = p->table_nT;
    // workspace of one grid size's table chains (grids, descriptors, block
    // offsets and redo buffers), as upload_chains carves them
    const int teb = table_angle_bytes(p);
    auto table_chain_bytes = [&](int b) {
        const int64_t hg = round_up(half_grid_bytes(tg[b].nx, tg[b].ny, teb), 256);
        return nT * 2 * hg + redo_bytes(tg[b].nx, tg[b].ny, nT) +
               nT * (int64_t)(sizeof(ChainDesc) + sizeof(ChainState) + 8 + (kNumStarts + 1) * 8) + 4096;
    };
    for (size_t first = 0; first < missing.size();) {
        // as many grid sizes as fit (at least one: the workspace holds the largest)
        size_t last = first;
        int64_t need = 65536 + table_chain_bytes(missing[first]);
        while (last + 1 < missing.size() && need + table_chain_bytes(missing[last + 1]) <= ws_bytes)
            need += table_chain_bytes(missing[++last]);
        Carver cv{(char *)ws, ws_bytes};
        ChainSet cs;
        cs.fp64 = teb == 8;
        int64_t maxn = 0;
        for (size_t g = first; g <= last; ++g) {
            const int b = missing[g];
            const int64_t tnx = tg[b].nx, tny = tg[b].ny;
            maxn = std::max(maxn, tnx * tny);
            for (int k = 0; k < nT; ++k) {
                ChainDesc d;
                std::memset(&d, 0, sizeof d);
                if (!carve_chain(cv, d, (int)tnx, (int)tny, false, false, teb))
                    return fail(ctx, MPR_ERR_WORKSPACE, "workspace too small");
                d.image_id = kTableStream;
                d.chain = (uint32_t)k;
                d.P = tnx * tny;
                d.ngp = tnx * (tny - 1) + tny * (tnx - 1);
                cs.desc.push_back(d);
                cs.state.push_back(fresh_state(Tg[k], PH_TABLE));
                cs.offset.push_back(0);
            }
        }
        int rc = upload_chains(ctx, cs, cv, stream, p->q);
        if (rc) return rc;
        launch_init(stream, cs, nullptr, nullptr, nullptr, 0u, 1);
        HIP_TRY(ctx, hipGetLastError());
        rc = run_chains(ctx, cs, p, stream, (int64_t)p->table_burn + p->table_meas, 50, true);
        if (rc) return rc;
        HIP_TRY(ctx, hipMemcpyAsync(cs.state.data(), cs.d_state, cs.state.size() * sizeof(ChainState),
                                    hipMemcpyDeviceToHost, stream));
        HIP_TRY(ctx, hipStreamSynchronize(stream));
        for (size_t g = first; g <= last; ++g) {
            std::vector<double> ope(nT);
            for (int k = 0; k < nT; ++k) ope[k] = cs.state[(g - first) * nT + k].e_sum / (double)p->table_meas;
            ctx->tables.emplace(key_of(missing[g]), ope);
        }
        first = last + 1;
    }
    for (int b = 0; b < n; ++b) {
        int cl = 0;
        T_hat[b] = invert_table(Tg, ctx->tables.at(key_of(b)), e_s[b], &cl);
        if (t_clamped) t_clamped[b] = cl;
    }
    return MPR_OK;
}

// mpr_simulate on the workspace ws (the caller's, checked as device memory,
// or this device's static workspace, `caller_ws` false); `graphs` false
// launches every sweep directly.
static int32_t simulate_call(mpr_ctx *ctx, const mpr_image *imgs, int32_t n, const float *phi,
                             const uint8_t *sampled, const double *T_hat, const mpr_params *p,
                             const float *phi_init, void *ws, int64_t ws_bytes, float *phi_sum, float *phi_m2,
                             float *phi_states, mpr_chain_stats *stats, void *stream_, bool caller_ws, bool graphs)
{
    if (!ctx) return MPR_ERR_ARG;
    if (!valid_images(imgs, n) || !valid_params(p) || !phi || !sampled || !T_hat || !phi_sum)
        return fail(ctx, MPR_ERR_ARG, "simulate: invalid argument");
    if (int rc = mpr_check_device(ctx, "simulate",
                                  {{"phi", phi}, {"sampled", sampled}, {"phi_init", phi_init},
                                   {"workspace", caller_ws ? ws : nullptr}, {"phi_sum", phi_sum},
                                   {"phi_m2", phi_m2}, {"phi_states", phi_states}}))
        return rc;
    if (phi_m2 && p->K > 1 && !p->spread)
        return fail(ctx, MPR_ERR_ARG, "simulate: phi_m2 with K > 1 needs params.spread = 1");
    if (phi_init && p->K < p->warm_min_states)
        return fail(ctx, MPR_ERR_ARG,
                    "simulate: a warm start (phi_init) needs K >= warm_min_states = %d equilibrium states per "
                    "chain (K = %d): every chain starts from the same angles",
                    p->warm_min_states, p->K);
    for (int b = 0; b < n; ++b)
        if (!(T_hat[b] > 0.0) || !std::isfinite(T_hat[b])) return fail(ctx, MPR_ERR_ARG, "image %d: bad T_hat", b);
    if (!ws || ws_bytes < sim_bytes(imgs, n, p)) return fail(ctx, MPR_ERR_WORKSPACE, "workspace too small");
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    hipStream_t stream = (hipStream_t)stream_;
    // gap counts (host needs them for the acceptance ratio): from the mask
    // via a device reduction would need scratch; count with the e_s-style
    // partials instead, reusing the map kernel's layout.
    Carver cv{(char *)ws, ws_bytes};
    // the run header: checked before a resumed run continues; a fresh run
    // marks the workspace as not resumable until it stops at sweep_limit
    RunHeader *d_hdr = (RunHeader *)cv.take(kRunHeaderBytes);
    const uint64_t key = run_key(imgs, n, p, T_hat);
    const bool resume = p->resume != 0;
    RunHeader hdr{kRunMagic, key, sim_bytes(imgs, n, p), n * p->R, 0};
    if (resume) {
        RunHeader old;
        HIP_TRY(ctx, hipMemcpyAsync(&old, d_hdr, sizeof old, hipMemcpyDeviceToHost, stream));
        HIP_TRY(ctx, hipStreamSynchronize(stream));
        if (old.magic != hdr.magic || old.key != hdr.key || old.bytes != hdr.bytes || old.n_chains != hdr.n_chains ||
            old.state != 1)
            return fail(ctx, MPR_ERR_ARG,
                        "simulate: resume needs a workspace holding a run stopped at sweep_limit with the same "
                        "images, parameters and temperatures");
    }
    // a call that fails leaves no run to resume: not the one the workspace held
    // before a fresh call (which may have written over it by then), nor one
    // whose sweeps were cut off
    HeaderGuard guard{resume ? nullptr : d_hdr, hdr, stream};
    ImgDev *d_img = (ImgDev *)cv.take(n * (int64_t)sizeof(ImgDev));
    std::vector<ImgDev> hi;
    ImgArgs img;
    if (int rc = image_args(ctx, stream, imgs, n, hi, d_img, img)) return rc;
    std::vector<int64_t> gaps(n, 0);
    {
        // count gaps with the map reduction on a constant z
        char *sp = (char *)ctx->scratch + kVarOffset;
        float *pmin = (float *)sp;
        int mb = 1;  // partial blocks per image (the counts are exact for any number)
        for (int b = 0; b < n; ++b) mb = std::max(mb, minmax_blocks((int64_t)hi[b].nx * hi[b].ny));
        mb = (int)std::max<int64_t>(1, std::min<int64_t>(mb, ((int64_t)kScratchBytes - kVarOffset - 512) / (24 * (int64_t)n)));
        float *pmax = pmin + (int64_t)n * mb;
        unsigned long long *pcnt = (unsigned long long *)(pmax + (int64_t)n * mb);
        unsigned int *pbad = (unsigned int *)(pcnt + (int64_t)n * mb);
        if ((int64_t)n * mb * 24 + 512 > (int64_t)kScratchBytes - kVarOffset)
            return fail(ctx, MPR_ERR_ARG, "too many images in one call");
        // map_minmax counts sampled sites of finite value; phi is finite.  The
        // counts go straight into pinned host memory where they fit.
        const int64_t cnt_bytes = (int64_t)n * mb * 8;
        std::vector<char> big;
        unsigned long long *hc = (unsigned long long *)stage_for(ctx, cnt_bytes, big);
        const bool direct = big.empty();
        hipLaunchKernelGGL(map_minmax_kernel, dim3(mb, n), dim3(kBlock), 0, stream, img, phi, sampled, pmin,
                           pmax, direct ? hc : pcnt, pbad);
        HIP_TRY(ctx, hipGetLastError());
        if (!direct) HIP_TRY(ctx, hipMemcpyAsync(hc, pcnt, (size_t)cnt_bytes, hipMemcpyDeviceToHost, stream));
        HIP_TRY(ctx, hipStreamSynchronize(stream));
        for (int b = 0; b < n; ++b) {
            unsigned long long c = 0;
            for (int k = 0; k < mb; ++k) c += hc[(size_t)b * mb + k];
            gaps[b] = (int64_t)imgs[b].nx * imgs[b].ny - (int64_t)c;
        }
    }
    ChainSet cs;
    for (int b = 0; b < n; ++b) {
        const int nx = imgs[b].nx, ny = imgs[b].ny;
        if ((int64_t)nx * ny < 2) return fail(ctx, MPR_ERR_DEGENERATE, "image %d: one site", b);
        for (int r = 0; r < p->R; ++r) {
            ChainDesc d;
            std::memset(&d, 0, sizeof d);
            if (!carve_chain(cv, d, nx, ny, p->K > 1, p->spread != 0, p->fp64 ? 8 : 4, !p->fp64))
                return fail(ctx, MPR_ERR_WORKSPACE, "workspace too small");
            d.image_id = imgs[b].id;
            d.chain = (uint32_t)r;
            d.P = gaps[b];
            d.ngp = (int64_t)nx * (ny - 1) + (int64_t)ny * (nx - 1);
            cs.desc.push_back(d);
            int phase = PH_RELAX;
            if (d.P == 0) phase = PH_DONE;
            else if (p->fixed_relax == 0) phase = p->K > 0 ? PH_EQ : PH_DONE;
            ChainState st = fresh_state(T_hat[b], phase);
            st.eq_left = p->K;
            if (phase == PH_EQ && !p->eq_a_mode) st.a_cur = 1.0;
            cs.state.push_back(st);
            cs.offset.push_back(imgs[b].offset);
        }
    }
    cs.fp64 = p->fp64 != 0;
    cs.K = p->K;
    if (phi_states && p->K > 0) {
        cs.states_out = phi_states;
        for (int b = 0; b < n; ++b)
            cs.states_n_total = std::max(cs.states_n_total, imgs[b].offset + (int64_t)imgs[b].nx * imgs[b].ny);
    }
    int rc = upload_chains(ctx, cs, cv, stream, p->q, resume);
    if (rc) return rc;
    int64_t maxn = 0;
    for (int b = 0; b < n; ++b) maxn = std::max(maxn, (int64_t)imgs[b].nx * imgs[b].ny);
    if (!resume) {
        launch_init(stream, cs, phi, sampled, phi_init, p->seed, 0, hdr, d_hdr);
        HIP_TRY(ctx, hipGetLastError());
    }
    // sweeps left to the run's cap (a resumed run has done `swept` of them),
    // and to this call's sweep_limit
    const int64_t relax_cap = p->fixed_relax >= 0 ? p->fixed_relax : (int64_t)p->i_max + 1;
    int64_t swept = 0;
    for (const auto &st : cs.state) swept = std::max<int64_t>(swept, (int64_t)st.sweep);
    int64_t limit = std::max<int64_t>(1, relax_cap + p->K + 1 - swept);
    if (p->sweep_limit > 0) limit = std::min<int64_t>(limit, p->sweep_limit);
    guard.d_hdr = d_hdr;
    rc = run_chains(ctx, cs, p, stream, limit, p->n_f, false, graphs, p->sweep_limit > 0);
    const bool incomplete = rc == MPR_INCOMPLETE;
    if (rc && !incomplete) return rc;
    guard.d_hdr = nullptr;
    if (incomplete || resume) {
        // resumable while chains are running, not once the run is finished
        hdr.state = incomplete ? 1 : 0;
        HIP_TRY(ctx, hipMemcpyAsync(d_hdr, &hdr, sizeof hdr, hipMemcpyHostToDevice, stream));
    }
    if (!incomplete) {  // an incomplete run writes no outputs, only its statistics so far
        if (cs.fp64)
            hipLaunchKernelGGL(finalize_fp64_kernel, dim3(blocks_for(maxn, 4096), n), dim3(kBlock), 0, stream,
                               cs.d_desc, img, p->R, p->K, sampled, phi_sum, phi_m2);
        else
            hipLaunchKernelGGL(finalize_kernel, dim3(blocks_for(maxn, 4096), n), dim3(kBlock), 0, stream,
                               cs.d_desc, img, p->R, p->K, sampled, phi_sum, phi_m2);
        HIP_TRY(ctx, hipGetLastError());
    }
    std::vector<char> big;
    const ChainState *final_state = nullptr;
    if (stats) {
        const int64_t bytes = (int64_t)(cs.state.size() * sizeof(ChainState));
        char *h = stage_for(ctx, bytes, big);
        HIP_TRY(ctx, hipMemcpyAsync(h, cs.d_state, (size_t)bytes, hipMemcpyDeviceToHost, stream));
        final_state = (const ChainState *)h;
    }
    HIP_TRY(ctx, hipStreamSynchronize(stream));
    if (stats) {
        for (size_t c = 0; c < cs.state.size(); ++c) {
            const ChainState &s = final_state[c];
            stats[c].relax_sweeps = s.relax_sweeps;
            stats[c].not_converged = s.not_converged;
            stats[c].a_final = s.a_relax;
            stats[c].A_last = s.A_last;
            stats[c].k_last = s.k;
        }
    }
    return incomplete ? MPR_INCOMPLETE : MPR_OK;
}

int32_t mpr_simulate(mpr_ctx *ctx, const mpr_image *imgs, int32_t n, const float *phi, const uint8_t *sampled,
                     const double *T_hat, const mpr_params *p, const float *phi_init, void *ws, int64_t ws_bytes,
                     float *phi_sum, float *phi_m2, float *phi_states, mpr_chain_stats *stats, void *stream_)
{
    return simulate_call(ctx, imgs, n, phi, sampled, T_hat, p, phi_init, ws, ws_bytes, phi_sum, phi_m2, phi_states,
                         stats, stream_, true, true);
}

int32_t mpr_simulate_noalloc(mpr_ctx *ctx, const mpr_image *imgs, int32_t n, const float *phi,
                             const uint8_t *sampled, const double *T_hat, const mpr_params *p,
                             const float *phi_init, float *phi_sum, float *phi_m2, float *phi_states,
                             mpr_chain_stats *stats, void *stream_)
{
    if (!ctx) return MPR_ERR_ARG;
    if (!valid_images(imgs, n) || !valid_params(p))
        return fail(ctx, MPR_ERR_ARG, "simulate_noalloc: invalid argument");
    if (!ctx->static_ws)
        return fail(ctx, MPR_ERR_HIP, "simulate_noalloc: no static workspace on device %d", ctx->device);
    const int64_t need = sim_bytes(imgs, n, p);
    if (need > kStaticWorkspaceBytes)
        return fail(ctx, MPR_ERR_WORKSPACE,
                    "simulate_noalloc: this batch needs %lld workspace bytes, the static workspace holds %lld "
                    "(use mpr_simulate with a workspace of mpr_workspace_size bytes)",
                    (long long)need, (long long)kStaticWorkspaceBytes);
    return simulate_call(ctx, imgs, n, phi, sampled, T_hat, p, phi_init, ctx->static_ws, kStaticWorkspaceBytes,
                         phi_sum, phi_m2, phi_states, stats, stream_, false, false);
}

int64_t mpr_simulate_noalloc_max_bytes(void) { return kStaticWorkspaceBytes; }

int32_t mpr_predict(mpr_ctx *ctx, const mpr_image *imgs, int32_t n, const float *z, const uint8_t *sampled,
                    const float *phi_sum, const double *zmin_zmax, int32_t M, float *z_hat, void *stream_)
{
    if (!ctx) return MPR_ERR_ARG;
    if (!valid_images(imgs, n) || !z || !sampled || !phi_sum || !zmin_zmax || !z_hat || M < 1)
        return fail(ctx, MPR_ERR_ARG, "predict: invalid argument");
    if (int rc = mpr_check_device(ctx, "predict",
                                  {{"z", z}, {"sampled", sampled}, {"phi_sum", phi_sum}, {"z_hat", z_hat}}))
        return rc;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    hipStream_t stream = (hipStream_t)stream_;
    const int64_t need = round_up((int64_t)n * sizeof(ImgDev), 256) + (int64_t)n * 16;
    if (need > (int64_t)kScratchBytes - kVarOffset) return fail(ctx, MPR_ERR_ARG, "too many images in one call");
    char *sp = (char *)ctx->scratch + kVarOffset;
    ImgDev *d_img = (ImgDev *)sp;
    double *d_zmm = (double *)(sp + round_up((int64_t)n * sizeof(ImgDev), 256));
    int64_t maxn = 0;
    for (int b = 0; b < n; ++b) maxn = std::max(maxn, (int64_t)imgs[b].nx * imgs[b].ny);
    std::vector<ImgDev> hi;
    ImgArgs img;
    RangeArgs range;
    if (int rc = image_args(ctx, stream, imgs, n, hi, d_img, img)) return rc;
    if (int rc = range_args(ctx, stream, zmin_zmax, n, d_zmm, range)) return rc;
    hipLaunchKernelGGL(predict_kernel, dim3(blocks_for(maxn, 4096), n), dim3(kBlock), 0, stream, img, range, M, z,
                       sampled, phi_sum, z_hat);
    HIP_TRY(ctx, hipGetLastError());
    // the host arrays above must outlive the copies
    HIP_TRY(ctx, hipStreamSynchronize(stream));
    return MPR_OK;
}

int32_t mpr_quantiles(mpr_ctx *ctx, const mpr_image *imgs, int32_t n, const float *z, const uint8_t *sampled,
                      const float *phi_states, int32_t M, const double *probs, int32_t nq, const double *zmin_zmax,
                      float *z_q, void *stream_)
{
    if (!ctx) return MPR_ERR_ARG;
    if (!valid_images(imgs, n) || !z || !sampled || !phi_states || !probs || !zmin_zmax || !z_q || M < 1 ||
        M > kMaxQuantileStates || nq < 1 || nq > kMaxProbs)
        return fail(ctx, MPR_ERR_ARG, "quantiles: invalid argument (1 <= M <= %d, 1 <= nq <= 64)",
                    kMaxQuantileStates);
    for (int k = 0; k < nq; ++k)
        if (!(probs[k] >= 0.0 && probs[k] <= 1.0)) return fail(ctx, MPR_ERR_ARG, "quantiles: p outside [0, 1]");
    if (int rc = mpr_check_device(ctx, "quantiles",
                                  {{"z", z}, {"sampled", sampled}, {"phi_states", phi_states}, {"z_q", z_q}}))
        return rc;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    hipStream_t stream = (hipStream_t)stream_;
    const int64_t img_bytes = round_up((int64_t)n * sizeof(ImgDev), 256);
    const int64_t need = img_bytes + round_up((int64_t)n * 16, 256) + nq * 8;
    if (need > (int64_t)kScratchBytes - kVarOffset) return fail(ctx, MPR_ERR_ARG, "too many images in one call");
    char *sp = (char *)ctx->scratch + kVarOffset;
    ImgDev *d_img = (ImgDev *)sp;
    double *d_zmm = (double *)(sp + img_bytes);
    std::vector<ImgDev> hi;
    int64_t maxn = 0, n_total = 0;
    for (int b = 0; b < n; ++b) {
        maxn = std::max(maxn, (int64_t)imgs[b].nx * imgs[b].ny);
        n_total = std::max(n_total, imgs[b].offset + (int64_t)imgs[b].nx * imgs[b].ny);
    }
    ImgArgs img;
    RangeArgs range;
    ProbArgs pr;
    if (int rc = image_args(ctx, stream, imgs, n, hi, d_img, img)) return rc;
    if (int rc = range_args(ctx, stream, zmin_zmax, n, d_zmm, range)) return rc;
    std::memset(&pr, 0, sizeof pr);
    std::memcpy(pr.v, probs, (size_t)nq * 8);
    // the smallest network that holds M states
    using Launch = void (*)(hipStream_t, int64_t, int, const ImgArgs &, const RangeArgs &, const ProbArgs &, int,
                            const float *, const uint8_t *, const float *, int, int64_t, float *);
    static constexpr Launch kNets[16] = {
        launch_quantiles<8, false>,   launch_quantiles<16, false>,  launch_quantiles<24, false>,
        launch_quantiles<32, false>,  launch_quantiles<40, false>,  launch_quantiles<48, false>,
        launch_quantiles<56, false>,  launch_quantiles<64, false>,  launch_quantiles<72, false>,
        launch_quantiles<80, false>,  launch_quantiles<88, false>,  launch_quantiles<96, false>,
        launch_quantiles<104, false>, launch_quantiles<112, false>, launch_quantiles<120, false>,
        launch_quantiles<128, false>};
    (M <= 128 ? kNets[(M - 1) / 8] : launch_quantiles<128, true>)(stream, maxn, n, img, range, pr, nq, z, sampled,
                                                                   phi_states, M, n_total, z_q);
    HIP_TRY(ctx, hipGetLastError());
    HIP_TRY(ctx, hipStreamSynchronize(stream));
    return MPR_OK;
}

int32_t mpr_spread(mpr_ctx *ctx, const mpr_image *imgs, int32_t n, const uint8_t *sampled, const float *phi_m2,
                   const double *zmin_zmax, int32_t M, float *z_std, void *stream_)
{
    if (!ctx) return MPR_ERR_ARG;
    if (!valid_images(imgs, n) || !sampled || !phi_m2 || !zmin_zmax || !z_std || M < 1)
        return fail(ctx, MPR_ERR_ARG, "spread: invalid argument");
    if (int rc = mpr_check_device(ctx, "spread", {{"sampled", sampled}, {"phi_m2", phi_m2}, {"z_std", z_std}}))
        return rc;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    hipStream_t stream = (hipStream_t)stream_;
    const int64_t need = round_up((int64_t)n * sizeof(ImgDev), 256) + (int64_t)n * 16;
    if (need > (int64_t)kScratchBytes - kVarOffset) return fail(ctx, MPR_ERR_ARG, "too many images in one call");
    char *sp = (char *)ctx->scratch + kVarOffset;
    ImgDev *d_img = (ImgDev *)sp;
    double *d_zmm = (double *)(sp + round_up((int64_t)n * sizeof(ImgDev), 256));
    int64_t maxn = 0;
    for (int b = 0; b < n; ++b) maxn = std::max(maxn, (int64_t)imgs[b].nx * imgs[b].ny);
    std::vector<ImgDev> hi;
    ImgArgs img;
    RangeArgs range;
    if (int rc = image_args(ctx, stream, imgs, n, hi, d_img, img)) return rc;
    if (int rc = range_args(ctx, stream, zmin_zmax, n, d_zmm, range)) return rc;
    hipLaunchKernelGGL(spread_kernel, dim3(blocks_for(maxn, 4096), n), dim3(kBlock), 0, stream, img, range, M,
                       sampled, phi_m2, z_std);
    HIP_TRY(ctx, hipGetLastError());
    HIP_TRY(ctx, hipStreamSynchronize(stream));
    return MPR_OK;
}

// Workspace of mpr_select_q: four per-site buffers of the image and the
// largest simulation/temperature workspace over the candidate q.
int64_t select_q_bytes(const mpr_image *img, const mpr_params *p, const double *q_grid, int nq)
{
    const int64_t n = (int64_t)img->nx * img->ny;
    mpr_image im0 = *img;
    im0.offset = 0;
    int64_t best = 0;
    for (int k = 0; k < nq; ++k) {
        mpr_params pk = *p;
        pk.q = q_grid[k];
        pk.fp64 = q_grid[k] == 0.5 ? p->fp64 : 1;
        if (!valid_params(&pk)) return -1;
        best = std::max(best, std::max(sim_bytes(&im0, 1, &pk), table_bytes(&im0, 1, &pk)));
    }
    return best + round_up(n, 256) + 3 * round_up(4 * n, 256) + 1024;
}

int64_t mpr_select_q_workspace_size(const mpr_image *img, const mpr_params *p, const double *q_grid, int32_t nq)
{
    if (!valid_images(img, 1) || !p || !q_grid || nq < 1) return -1;
    return select_q_bytes(img, p, q_grid, nq);
}

int32_t mpr_select_q(mpr_ctx *ctx, const mpr_image *img, const float *z, const uint8_t *sampled, const mpr_params *p,
                     const double *q_grid, int32_t nq, double holdout, void *ws, int64_t ws_bytes, double *val_mae,
                     double *T_hat, double *q_best, void *stream_)
{
    if (!ctx) return MPR_ERR_ARG;
    if (!valid_images(img, 1) || !z || !sampled || !p || !q_grid || nq < 1 || nq > 64 || !(holdout > 0.0) ||
        !(holdout < 1.0) || !val_mae || !q_best || p->K < 1)
        return fail(ctx, MPR_ERR_ARG, "select_q: invalid argument");
    const int64_t need = select_q_bytes(img, p, q_grid, nq);
    if (need < 0) return fail(ctx, MPR_ERR_ARG, "select_q: a candidate q is outside (0, 1/2]");
    if (!ws || ws_bytes < need) return fail(ctx, MPR_ERR_WORKSPACE, "workspace too small");
    if (int rc = mpr_check_device(ctx, "select_q", {{"z", z}, {"sampled", sampled}, {"workspace", ws}})) return rc;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    hipStream_t stream = (hipStream_t)stream_;
    const int64_t n = (int64_t)img->nx * img->ny;
    mpr_image im0 = *img;
    im0.offset = 0;
    const float *zi = z + img->offset;
    const uint8_t *si = sampled + img->offset;
    // per-site buffers first, the calls' workspace after them
    const int64_t head = round_up(n, 256) + 3 * round_up(4 * n, 256);
    uint8_t *fit = (uint8_t *)ws;
    float *phi = (float *)((char *)ws + round_up(n, 256));
    float *psum = (float *)((char *)phi + round_up(4 * n, 256));
    float *zhat = (float *)((char *)psum + round_up(4 * n, 256));
    void *iws = (char *)ws + head;
    const int64_t inner = ws_bytes - head;
    hipLaunchKernelGGL(holdout_kernel, dim3(blocks_for(n, 2048)), dim3(kBlock), 0, stream, img->nx, img->ny, si,
                       (uint32_t)p->seed, (uint32_t)(p->seed >> 32), holdout, fit);
    HIP_TRY(ctx, hipGetLastError());
    double zmm[2];
    int rc = mpr_map_to_angles(ctx, &im0, 1, zi, fit, phi, zmm, stream);
    if (rc) return rc;
    double *d_ps = (double *)((char *)ctx->scratch + kVarOffset);
    unsigned long long *d_pc = (unsigned long long *)(d_ps + kHoldoutBlocks);
    int best = -1;
    for (int k = 0; k < nq; ++k) {
        mpr_params pk = *p;
        pk.q = q_grid[k];
        pk.fp64 = q_grid[k] == 0.5 ? p->fp64 : 1;
        double e_s = 0.0, T = 0.0;
        rc = mpr_estimate_temperature(ctx, &im0, 1, phi, fit, &pk, iws, inner, &e_s, &T, nullptr, stream);
        if (rc) return rc;
        rc = mpr_simulate(ctx, &im0, 1, phi, fit, &T, &pk, nullptr, iws, inner, psum, nullptr, nullptr, nullptr,
                          stream);
        if (rc) return rc;
        rc = mpr_predict(ctx, &im0, 1, zi, fit, psum, zmm, pk.R * pk.K, zhat, stream);
        if (rc) return rc;
        hipLaunchKernelGGL(holdout_error_kernel, dim3(kHoldoutBlocks), dim3(kBlock), 0, stream, n, zi, si, fit,
                           zhat, d_ps, d_pc);
        HIP_TRY(ctx, hipGetLastError());
        double hs[kHoldoutBlocks];
        unsigned long long hc[kHoldoutBlocks];
        HIP_TRY(ctx, hipMemcpyAsync(hs, d_ps, sizeof hs, hipMemcpyDeviceToHost, stream));
        HIP_TRY(ctx, hipMemcpyAsync(hc, d_pc, sizeof hc, hipMemcpyDeviceToHost, stream));
        HIP_TRY(ctx, hipStreamSynchronize(stream));
        double sum = 0.0;
        unsigned long long cnt = 0;
        for (int b = 0; b < kHoldoutBlocks; ++b) {
            sum += hs[b];
            cnt += hc[b];
        }
        if (cnt == 0) return fail(ctx, MPR_ERR_DEGENERATE, "select_q: no sample held out");
        val_mae[k] = sum / (double)cnt;
        if (T_hat) T_hat[k] = T;
        // smallest error; on a tie the larger q
        if (best < 0 || val_mae[k] < val_mae[best] || (val_mae[k] == val_mae[best] && q_grid[k] > q_grid[best]))
            best = k;
    }
    *q_best = q_grid[best];
    return MPR_OK;
}

int32_t mpr_profile_enable(mpr_ctx *ctx, int32_t on)
{
    if (!ctx) return MPR_ERR_ARG;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    ctx->profile = on != 0;
    ctx->prof_ms = 0.0;
    ctx->prof_launches = 0;
    HIP_TRY(ctx, hipMemset((char *)ctx->scratch + kWorkOffset, 0, 3 * sizeof(unsigned long long)));
    return MPR_OK;
}

int32_t mpr_profile_read(mpr_ctx *ctx, mpr_profile *out)
{
    if (!ctx || !out) return MPR_ERR_ARG;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    unsigned long long w[3] = {0, 0, 0};
    HIP_TRY(ctx, hipMemcpy(w, (char *)ctx->scratch + kWorkOffset, sizeof w, hipMemcpyDeviceToHost));
    out->sweep_kernel_ms = ctx->prof_ms;
    out->sweep_launches = ctx->prof_launches;
    out->last_tile = ctx->last_tile;
    out->reserved = 0;
    out->chain_sweeps = (int64_t)w[0];
    out->site_updates = (int64_t)w[1];
    out->useful_bytes = (double)w[2];
    return MPR_OK;
}

// ------------------------------------------------------------ diagnostics

int32_t mpr_diag_philox(mpr_ctx *ctx, const uint32_t *ctr, uint64_t seed, int64_t n, uint32_t *out, void *stream_)
{
    if (!ctx) return MPR_ERR_ARG;
    if (!ctr || !out || n < 0) return fail(ctx, MPR_ERR_ARG, "diag_philox: invalid argument");
    if (int rc = mpr_check_device(ctx, "diag_philox", {{"ctr", ctr}, {"out", out}})) return rc;
    if (n == 0) return MPR_OK;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    hipStream_t stream = (hipStream_t)stream_;
    hipLaunchKernelGGL(philox_kernel, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, stream, ctr,
                       (uint32_t)seed, (uint32_t)(seed >> 32), n, out);
    HIP_TRY(ctx, hipGetLastError());
    HIP_TRY(ctx, hipStreamSynchronize(stream));
    return MPR_OK;
}

int32_t mpr_diag_half_sweep(mpr_ctx *ctx, int32_t nx, int32_t ny, float *phi, const uint8_t *sampled, int32_t colour,
                            double T, double a, double q, uint64_t seed, uint32_t sweep, uint32_t chain,
                            uint32_t stream_id, int32_t mode, int32_t tile, uint8_t *flags, int64_t *accepted,
                            double *bond_energy, void *stream_)
{
    if (!ctx) return MPR_ERR_ARG;
    const int v = tile ? shape_of(tile) : kDefaultShape;
    if (nx < 1 || ny < 1 || (int64_t)nx * ny < 2 || half_grid_bytes(nx, ny) >= ((int64_t)1 << 32) || !phi ||
        !sampled || (colour != 0 && colour != 1) || !(T > 0) || !(a > 0) || q != 0.5 || (mode != 0 && mode != 1) ||
        v < 0)
        return fail(ctx, MPR_ERR_ARG, "diag_half_sweep: invalid argument");
    if (int rc = mpr_check_device(ctx, "diag_half_sweep", {{"phi", phi}, {"sampled", sampled}, {"flags", flags}}))
        return rc;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    hipStream_t stream = (hipStream_t)stream_;
    const int64_t hg = half_grid_bytes(nx, ny);
    const int64_t bytes = 2 * round_up(hg, 256) + 8192 + redo_bytes(nx, ny, 1);
    void *buf = nullptr;
    HIP_TRY(ctx, hipMalloc(&buf, bytes));
    Carver cv{(char *)buf, bytes};
    ChainSet cs;
    ChainDesc d;
    std::memset(&d, 0, sizeof d);
    carve_chain(cv, d, nx, ny, false);
    d.image_id = stream_id;
    d.chain = chain;
    d.P = 1;
    d.ngp = (int64_t)nx * (ny - 1) + (int64_t)ny * (nx - 1);
    cs.desc.push_back(d);
    ChainState st = fresh_state(T, PH_RELAX);
    st.sweep = sweep;
    st.a_cur = a;
    cs.state.push_back(st);
    cs.offset.push_back(0);
    int rc = upload_chains(ctx, cs, cv, stream, q);
    if (!rc) rc = clear_redo(ctx, cs, stream);
    if (rc) {
        (void)hipFree(buf);
        return rc;
    }
    const int64_t nsite = (int64_t)nx * ny;
    // the gap values of phi are the starting state
    launch_init(stream, cs, phi, sampled, phi, 0u, 0);
    if (flags) (void)hipMemsetAsync(flags, 0, nsite, stream);
    const SweepConsts sc = make_sc(q, seed);
    const dim3 grid((unsigned)cs.total_blocks[v]);
    const Shape sh = kShapes[v];
    const Redo rd = cs.redo;
    if (sh.fused) {
        launch_tile<true>(stream, cs, v, colour + 1, sc, mode, flags);
    } else if (sh.compact) {
        if (sh.rows == 2)
            hipLaunchKernelGGL((half_sweep_compact_kernel<true, 2>), grid, dim3(kBlock), 0, stream, cs.d_desc,
                               cs.d_state, block_map(cs, v), colour, sc, mode, rd, flags);
        else if (sh.rows == 4)
            hipLaunchKernelGGL((half_sweep_compact_kernel<true, 4>), grid, dim3(kBlock), 0, stream, cs.d_desc,
                               cs.d_state, block_map(cs, v), colour, sc, mode, rd, flags);
        else
            hipLaunchKernelGGL((half_sweep_compact_kernel<true, 8>), grid, dim3(kBlock), 0, stream, cs.d_desc,
                               cs.d_state, block_map(cs, v), colour, sc, mode, rd, flags);
    } else {
        if (sh.rows == 1)
            hipLaunchKernelGGL((half_sweep_kernel<true, 1>), grid, dim3(kBlock), 0, stream, cs.d_desc, cs.d_state,
                               block_map(cs, v), colour, sc, mode, rd, flags);
        else if (sh.rows == 2)
            hipLaunchKernelGGL((half_sweep_kernel<true, 2>), grid, dim3(kBlock), 0, stream, cs.d_desc, cs.d_state,
                               block_map(cs, v), colour, sc, mode, rd, flags);
        else if (sh.rows == 4)
            hipLaunchKernelGGL((half_sweep_kernel<true, 4>), grid, dim3(kBlock), 0, stream, cs.d_desc, cs.d_state,
                               block_map(cs, v), colour, sc, mode, rd, flags);
        else
            hipLaunchKernelGGL((half_sweep_kernel<true, 8>), grid, dim3(kBlock), 0, stream, cs.d_desc, cs.d_state,
                               block_map(cs, v), colour, sc, mode, rd, flags);
    }
    if (!sh.fused) launch_redo<true>(stream, cs, v, colour, sc, mode, flags);
    hipLaunchKernelGGL(unsplit_kernel, dim3(blocks_for(nsite, 2048)), dim3(kBlock), 0, stream, cs.d_desc, phi);
    ChainState out;
    (void)hipMemcpyAsync(&out, cs.d_state, sizeof out, hipMemcpyDeviceToHost, stream);
    hipError_t e1 = hipGetLastError();
    hipError_t e2 = hipStreamSynchronize(stream);
    (void)hipFree(buf);
    if (e1 != hipSuccess || e2 != hipSuccess)
        return fail(ctx, MPR_ERR_HIP, "diag_half_sweep: %s", hipGetErrorString(e1 != hipSuccess ? e1 : e2));
    if (accepted) *accepted = (int64_t)out.acc;
    if (bond_energy) *bond_energy = (double)out.e_fx * kEnergyUnit;
    return MPR_OK;
}

int32_t mpr_diag_half_sweep_fp64(mpr_ctx *ctx, int32_t nx, int32_t ny, double *phi, const uint8_t *sampled,
                                 int32_t colour, double T, double a, double q, uint64_t seed, uint32_t sweep,
                                 uint32_t chain, uint32_t stream_id, int32_t mode, int32_t tile, uint8_t *flags,
                                 int64_t *accepted, double *bond_energy, void *stream_)
{
    if (!ctx) return MPR_ERR_ARG;
    const int v = tile ? shape_of(tile) : kDefaultShape;
    if (nx < 1 || ny < 1 || (int64_t)nx * ny < 2 || half_grid_bytes(nx, ny) >= ((int64_t)1 << 32) || !phi ||
        !sampled || (colour != 0 && colour != 1) || !(T > 0) || !(a > 0) || !(q > 0.0 && q <= 0.5) ||
        (mode != 0 && mode != 1) || v < 0)
        return fail(ctx, MPR_ERR_ARG, "diag_half_sweep_fp64: invalid argument");
    if (int rc = mpr_check_device(ctx, "diag_half_sweep_fp64", {{"phi", phi}, {"sampled", sampled}, {"flags", flags}}))
        return rc;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    hipStream_t stream = (hipStream_t)stream_;
    const int64_t hg = half_grid_bytes(nx, ny, 8);
    const int64_t bytes = 2 * round_up(hg, 256) + 8192 + redo_bytes(nx, ny, 1);
    void *buf = nullptr;
    HIP_TRY(ctx, hipMalloc(&buf, bytes));
    Carver cv{(char *)buf, bytes};
    ChainSet cs;
    cs.fp64 = true;
    ChainDesc d;
    std::memset(&d, 0, sizeof d);
    carve_chain(cv, d, nx, ny, false, false, 8);
    d.image_id = stream_id;
    d.chain = chain;
    d.P = 1;
    d.ngp = (int64_t)nx * (ny - 1) + (int64_t)ny * (nx - 1);
    cs.desc.push_back(d);
    ChainState st = fresh_state(T, PH_RELAX);
    st.sweep = sweep;
    st.a_cur = a;
    cs.state.push_back(st);
    cs.offset.push_back(0);
    int rc = upload_chains(ctx, cs, cv, stream, q);
    if (rc) {
        (void)hipFree(buf);
        return rc;
    }
    (void)hipMemsetAsync(d.h[0], 0, hg, stream);
    (void)hipMemsetAsync(d.h[1], 0, hg, stream);
    const int64_t nsite = (int64_t)nx * ny;
    hipLaunchKernelGGL(split_fp64_kernel, dim3(blocks_for(nsite, 2048)), dim3(kBlock), 0, stream, cs.d_desc, phi,
                       sampled);
    if (flags) (void)hipMemsetAsync(flags, 0, nsite, stream);
    launch_half_fp64<true>(stream, cs, v, colour, make_sc(q, seed), mode, flags);
    hipLaunchKernelGGL(unsplit_fp64_kernel, dim3(blocks_for(nsite, 2048)), dim3(kBlock), 0, stream, cs.d_desc, phi);
    ChainState out;
    (void)hipMemcpyAsync(&out, cs.d_state, sizeof out, hipMemcpyDeviceToHost, stream);
    hipError_t e1 = hipGetLastError();
    hipError_t e2 = hipStreamSynchronize(stream);
    (void)hipFree(buf);
    if (e1 != hipSuccess || e2 != hipSuccess)
        return fail(ctx, MPR_ERR_HIP, "diag_half_sweep_fp64: %s", hipGetErrorString(e1 != hipSuccess ? e1 : e2));
    if (accepted) *accepted = (int64_t)out.acc;
    if (bond_energy) *bond_energy = (double)out.e_fx * kEnergyUnit64;
    return MPR_OK;
}

int32_t mpr_diag_copy(mpr_ctx *ctx, const void *src, void *dst, int64_t bytes, void *stream_)
{
    if (!ctx) return MPR_ERR_ARG;
    if (!src || !dst || bytes < 0 || bytes % 16 != 0 || ((uintptr_t)src | (uintptr_t)dst) % 16 != 0)
        return fail(ctx, MPR_ERR_ARG, "diag_copy: invalid argument");
    if (int rc = mpr_check_device(ctx, "diag_copy", {{"src", src}, {"dst", dst}})) return rc;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    hipStream_t stream = (hipStream_t)stream_;
    const int64_t n = bytes / 16;
    if (n > 0)
        hipLaunchKernelGGL(copy_probe_kernel, dim3(blocks_for(n, 8192)), dim3(kBlock), 0, stream,
                           (const float4 *)src, (float4 *)dst, n);
    HIP_TRY(ctx, hipGetLastError());
    HIP_TRY(ctx, hipStreamSynchronize(stream));
    return MPR_OK;
}

int32_t mpr_diag_energy(mpr_ctx *ctx, int32_t nx, int32_t ny, const float *phi, double q, double *h_plus_ngp,
                        void *stream_)
{
    if (!ctx) return MPR_ERR_ARG;
    if (nx < 1 || ny < 1 || !phi || !h_plus_ngp || !(q > 0 && q <= 0.5))
        return fail(ctx, MPR_ERR_ARG, "diag_energy: invalid argument");
    if (int rc = mpr_check_device(ctx, "diag_energy", {{"phi", phi}})) return rc;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    hipStream_t stream = (hipStream_t)stream_;
    unsigned long long *d_e = (unsigned long long *)((char *)ctx->scratch + kEnergyOffset);
    HIP_TRY(ctx, hipMemsetAsync(d_e, 0, 8, stream));
    hipLaunchKernelGGL(grid_energy_kernel, dim3(blocks_for((int64_t)nx * ny, 2048)), dim3(kBlock), 0, stream, phi, nx,
                       ny, (float)q, d_e);
    HIP_TRY(ctx, hipGetLastError());
    unsigned long long e = 0;
    HIP_TRY(ctx, hipMemcpyAsync(&e, d_e, 8, hipMemcpyDeviceToHost, stream));
    HIP_TRY(ctx, hipStreamSynchronize(stream));
    *h_plus_ngp = (double)e * kEnergyUnit;
    return MPR_OK;
}

int32_t mpr_diag_sg_slope(mpr_ctx *ctx, const double *e, int32_t n, int32_t degree, double *slope)
{
    if (!ctx) return MPR_ERR_ARG;
    if (!e || !slope || n < 2 || n > kMaxFit || degree < 1 || degree >= n)
        return fail(ctx, MPR_ERR_ARG, "diag_sg_slope: invalid argument");
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    mpr_params p;
    mpr_default_params(&p);
    p.n_fit = n;
    p.sg_degree = degree;
    const CtlParams cp = make_ctl(&p);
    double *d = (double *)((char *)ctx->scratch + kSlopeOffset);
    HIP_TRY(ctx, hipMemcpy(d, e, n * 8, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(ring_slope_kernel, dim3(1), dim3(1), 0, 0, d, n, cp, d + kMaxFit);
    HIP_TRY(ctx, hipGetLastError());
    HIP_TRY(ctx, hipMemcpy(slope, d + kMaxFit, 8, hipMemcpyDeviceToHost));
    return MPR_OK;
}

}  // extern "C"
