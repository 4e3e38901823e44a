// Re-binning: neighbour-table rows, particle copies and the bodies of its
// three passes (described in k_rebin.hip).
#pragma once

#include "pic_dev.h"

namespace pic {

// The neighbour table of a simulation (built once on the host from the patch
// grid) holds per patch: the canonical key of each of the ND directions (the
// smallest direction reaching the same neighbour; -1 when the neighbour is the
// patch itself, i.e. the particle stays; ND when it leaves an open face),
// then the number of distinct source patches, the sources in ascending id and
// the key under which each source stages the particles it sends here.  Key ND
// also stands for a removed particle.
template <int ND>
__device__ __forceinline__ gptr_t<const int32_t> nb_row(const int32_t *nbt, int p)
{
    return glb(nbt) + (int64_t)p * nb_stride(ND);
}

template <typename T>
__device__ __forceinline__ void copy_particle(const SimDev<T> &S, int64_t from, int64_t to,
                                              bool from_stage, bool to_stage)
{
    T *fP = from_stage ? S.spos : S.pos, *fM = from_stage ? S.smom : S.mom;
    T *tP = to_stage ? S.spos : S.pos, *tM = to_stage ? S.smom : S.mom;
    const int64_t *fi = from_stage ? S.sid : S.id;
    int64_t *ti = to_stage ? S.sid : S.id;
    v4(tM)[to] = v4(fM)[from];
    if (S.pw == 4) {
        v4(tP)[to] = v4(fP)[from];  // (with the id)
    } else {
        v2(tP)[to] = v2(fP)[from];
        glb(ti)[to] = glb(fi)[from];
    }
}

// Count pass.  Each wave of the workgroup owns a contiguous range of the
// patch's slots and loads the destination codes of up to kU x 64 of them at
// once (one batch; a patch of at most waves x kU x 64 particles is one batch).
// It lists the batch's leavers in LDS in slot order (a ballot per 64 slots) and
// counts them per key with LDS atomics.  After one exchange of the per-wave
// counts every wave knows where its leavers go; it then takes its list 64
// leavers at a time, one per lane: the vacated slots are a plain copy of the
// list, the rank among the leavers of a key comes from one ballot per key
// present, and the particle loads of the 64 are in flight together.  The chain
// of these rounds bounds the pass (a ballot per key and 64 slots, twice, and the
// codes of a second batch fetched again took, us per step: 64 x 48 x 40 box
// 174 -> 156, 128 x 128 46 -> 43, 512 x 128 FP64 laser box 54 -> 48, 1024 x 1024
// 436 -> 426, 256 x 128 x 128 2276 -> 2242).
// threads of the count workgroup: 256 in 2-D (512 and 128 slower), and in 3-D
// one wave per patch where the patches fill the chip (about a hundred
// leavers per 8^3 patch; measured beside the field update, smaller workgroups
// keep more patches in flight), else 256 (one wave's walk of a patch is then
// the whole pass: 64 x 48 x 40 box, 240 patches, 85 against 29 us,
// measured before the list below)
constexpr int kRC = 256;
constexpr int kRC3 = 64;
constexpr int kRC3Patches = 2048;
constexpr int kU = 16;    // 64-slot chunks per batch of code loads
constexpr int kList = 64 * kU + 256;  // listed leavers of a wave (4 KB: 8 waves per SIMD fit)

template <int ND, int NWV>
struct CountSmem {
    uint8_t kb[256];              // code -> key + 1 (0: the particle stays)
    int wc[NWV][ND + 3];          // per wave: leavers of each key, then of all keys
    // per wave: listed leavers, slot (from the wave's first one, or in the batch) and key + 1
    uint16_t slot[NWV][kList];
    uint8_t key[NWV][kList];
};

// Leavers of patch p: per-key counts (kcnt, nleave), the vacated slots in
// ascending order (holes) and the staged copies of the leavers, grouped by
// destination key in slot order.  Called by every thread of a workgroup of
// NWV waves (contains barriers).  n and base are the patch's count and first
// slot, key (threads tid < ND) the canonical key of direction tid: the caller
// loads them together with its own checks, so that their latencies overlap,
// and the first codes are loaded before the key table is built.
template <typename T, int ND, int NWV>
__device__ __forceinline__ void count_patch(const SimDev<T> &S, int p, int n, int64_t base, int key,
                                            CountSmem<ND, NWV> &sm)
{
    constexpr int kKeys = ND + 1;  // ND direction keys + removed
    constexpr int kThreads = NWV * 64;
    // (NWV == 1: one wave per patch, synchronised by wave barriers only)
    const int tid = NWV == 1 ? (int)(threadIdx.x & 63) : (int)threadIdx.x;
    const int lane = threadIdx.x & 63, wave = NWV == 1 ? 0 : (int)(threadIdx.x >> 6);
    auto group_sync = [&]() {
        if constexpr (NWV == 1) __builtin_amdgcn_wave_barrier();
        else __syncthreads();
    };
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const gptr_t<const uint8_t> code = glb((const uint8_t *)S.code) + base;
    const int per = ((n + kThreads - 1) / kThreads) * 64;
    const int lo = min(n, wave * per), hi = min(n, lo + per);
    uint8_t t[kU];  // codes of a batch
    auto fetch = [&](int q0) {
        const gptr_t<const uint8_t> cp = code + q0 + lane;
        const int left = hi - q0 - lane;  // chunk u holds a slot while 64 u < left
#pragma unroll
        for (int u = 0; u < kU; ++u) t[u] = 64 * u < left ? cp[64 * u] : uint8_t(ND / 2);
    };
    // append the leavers of batch q0 to the list of m entries, slots counted
    // from `from`, and fetch the next batch; returns the entries then
    uint16_t *lslot = sm.slot[wave];
    uint8_t *lkey = sm.key[wave];
    auto compact = [&](int q0, int from, int m) {
        uint32_t cw[kU / 4];  // keys + 1, four 64-slot chunks per register
#pragma unroll
        for (int u = 0; u < kU; u += 4)
            cw[u / 4] = (uint32_t)sm.kb[t[u]] | ((uint32_t)sm.kb[t[u + 1]] << 8) |
                        ((uint32_t)sm.kb[t[u + 2]] << 16) | ((uint32_t)sm.kb[t[u + 3]] << 24);
        if (q0 + 64 * kU < hi) fetch(q0 + 64 * kU);
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (q0 + 64 * u >= hi) break;
            const int kc = (int)((cw[u / 4] >> (8 * (u % 4))) & 0xffu);
            const uint64_t b = __ballot(kc != 0);
            if (kc) {
                const int at = m + __popcll(b & lt);
                lslot[at] = (uint16_t)(q0 - from + 64 * u + lane);
                lkey[at] = (uint8_t)kc;
            }
            m += __popcll(b);
        }
        __builtin_amdgcn_wave_barrier();
        return m;
    };
    fetch(lo);
    for (int e = tid; e < 256; e += kThreads) {
        int kb = 0;
        if (e < ND) kb = key + 1;  // e == tid here (ND < kThreads)
        else if (e == kRemoved) kb = ND + 1;
        sm.kb[e] = (uint8_t)kb;
    }
    group_sync();

    // ---- walk 1: leavers per key in [lo, hi) ------------------------------
    int *wc = sm.wc[wave];
    if (lane <= kKeys) wc[lane] = 0;
    __builtin_amdgcn_wave_barrier();
    // the list of all batches is kept for walk 2 while it has room for
    // another batch and slots fit 16 bits
    bool kept = hi - lo <= 65536;
    int m = 0, all = 0;
    for (int q0 = lo; q0 < hi; q0 += 64 * kU) {
        if (!kept || m > kList - 64 * kU) {
            kept = false;
            m = 0;
        }
        const int m0 = m;
        m = compact(q0, kept ? lo : q0, m0);
        all += m - m0;
        for (int i = m0 + lane; i < m; i += 64) atomicAdd(&wc[lkey[i] - 1], 1);
        __builtin_amdgcn_wave_barrier();
    }
    if (lane == kKeys) wc[kKeys] = all;
    group_sync();

    // ---- starting points: lane k of wave w holds the staging slot of the
    // next key-k leaver of the wave (key offset + earlier waves), lane kKeys
    // the next hole index ---------------------------------------------------
    int run = 0, tot = 0;
    if (lane <= kKeys)
        for (int w = 0; w < NWV; ++w) {
            const int c = sm.wc[w][lane];
            run += w < wave ? c : 0;
            tot += c;
        }
    int incl = tot;
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) {
        const int y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane < kKeys) run += incl - tot;
    if (wave == 0 && lane <= kKeys) {
        if (lane < ND) glb(S.kcnt)[p * ND + lane] = tot;
        if (lane < kKeys) glb(S.kofs)[p * kKeys + lane] = run;  // wave 0: the key's offset
        if (lane == kKeys) glb(S.nleave)[p] = tot;
    }

    // ---- walk 2: list holes, copy staged leavers ---------------------------
    if (all > 0) {
        if (!kept) fetch(lo);
        for (int q0 = lo; q0 < hi; q0 += kept ? hi - lo : 64 * kU) {
            if (!kept) m = compact(q0, q0, 0);
            for (int e0 = 0; e0 < m; e0 += 64) {
                const bool has = e0 + lane < m;
                const int kc = has ? lkey[e0 + lane] : 0, k = has ? q0 + lslot[e0 + lane] : 0;
                const int h0 = __builtin_amdgcn_readlane(run, kKeys);
                if (has) glb(S.holes)[base + h0 + lane] = k;
                run += lane == kKeys ? min(64, m - e0) : 0;
                int dest = 0;
                uint64_t todo = __ballot(has);
                while (todo) {
                    const int kk = __builtin_amdgcn_readlane(kc, __ffsll((long long)todo) - 1);
                    const uint64_t b = __ballot(kc == kk);
                    const int r0 = __builtin_amdgcn_readlane(run, kk - 1);
                    if (kc == kk) dest = r0 + __popcll(b & lt);
                    run += lane == kk - 1 ? __popcll(b) : 0;
                    todo &= ~b;
                }
                if (has && kc != ND + 1) copy_particle(S, base + k, base + dest, false, true);
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    group_sync();
}

// Count pass over the patches of workgroup wg of nwg (NT threads).
template <typename T, int ND, int NT>
__device__ __forceinline__ void rebin_count_patches(const SimDev<T> *__restrict__ sims, int nsims,
                                                    const int *__restrict__ patch_prefix, int total, int wg,
                                                    int nwg)
{
    __shared__ CountSmem<ND, NT / 64> sm;
    for (int gp = wg; gp < total; gp += nwg) {
        const int s = find_sim(patch_prefix, nsims, gp);
        const SimDev<T> &S = sims[s];
        const int p = gp - patch_prefix[s];
        // the state the patch's count needs, loaded together
        const uint32_t active = glb(S.st)->active;
        const int moved = *glb(S.moved + p);
        const int n = glb(S.count)[p];
        const int64_t base = glb(S.off)[p];
        const int key = threadIdx.x < ND ? nb_row<ND>(S.nbt, p)[threadIdx.x] : 0;
        if (!active) continue;
        if (!moved) {
            // no particle of the patch changed patch or was removed: no leavers
            if (threadIdx.x < ND) glb(S.kcnt)[p * ND + threadIdx.x] = 0;
            if (threadIdx.x <= ND) glb(S.kofs)[p * (ND + 1) + threadIdx.x] = 0;
            if (threadIdx.x == 0) glb(S.nleave)[p] = 0;
            continue;
        }
        count_patch<T, ND, NT / 64>(S, p, n, base, key, sm);
    }
}

// Lanes that check one patch: one per possible source (26 or 8), so the
// counts of all sources are one round of loads instead of a serial walk, and
// the vacated slots are searched kCheckLanes + 1 parts at a time (64 x 48 x 40
// box 17 -> 6 us per launch, 4096 x 1024 laser box beside the field update
// 26 -> 15 us).
template <int ND>
constexpr int kCheckLanes = ND == kNDir3 ? 32 : 8;
// Check pass of one patch (wg: workgroup of 256 threads).
template <typename T, int ND>
__device__ __forceinline__ void rebin_check_patches(const SimDev<T> *__restrict__ sims, int nsims,
                                                    const int *__restrict__ patch_prefix, int total, int wg)
{
    constexpr int G = kCheckLanes<ND>;
    const int gp = (int)((wg * (int64_t)256 + threadIdx.x) / G);
    const int l = threadIdx.x % G;
    if (gp >= total) return;  // (the whole group)
    const int s = find_sim(patch_prefix, nsims, gp);
    const SimDev<T> &S = sims[s];
    const int q = gp - patch_prefix[s];
    const gptr_t<const int32_t> row = nb_row<ND>(S.nbt, q);
    const int i = min(l, ND - 2);  // (always an entry of the row)
    const uint32_t active = glb(S.st)->active;
    const int ns = row[ND], src = row[ND + 1 + i], key = row[2 * ND + i];
    const int n = glb(S.count)[q], L = glb(S.nleave)[q];
    const gptr_t<const int32_t> h = glb((const int32_t *)S.holes) + glb(S.off)[q];
    if (!active) return;
    int A = l < ns ? glb(S.kcnt)[src * ND + key] : 0;
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) A += __shfl_xor(A, o, G);
    const int np = n - L + A;
    // vacated slots below the new count (the list is ascending)
    int lo = 0, hi = L;
    while (lo < hi) {
        auto probe = [&](int j) { return lo + (int)((int64_t)(hi - lo) * (j + 1) / (G + 1)); };
        const uint64_t below = __ballot(h[probe(l)] < np) >> (threadIdx.x & 63 & ~(G - 1));
        const int c = __popcll(below & ((1ull << G) - 1));
        const int lo2 = c > 0 ? probe(c - 1) + 1 : lo;
        hi = c < G ? probe(c) : hi;
        lo = lo2;
    }
    if (l != 0) return;
    glb(S.newcount)[q] = np;
    glb(S.narrive)[q] = A;
    glb(S.nhole)[q] = lo;
    if (np > glb(S.cap)[q])
        __hip_atomic_fetch_or(&glb(S.st)->flags, kFlagPending, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Scatter pass over the patches of workgroup wg of nwg (NT threads).
template <typename T, int ND, int NT>
__device__ __forceinline__ void rebin_scatter_patches(const SimDev<T> *__restrict__ sims, int nsims,
                                                      const int *__restrict__ patch_prefix, int total, int wg,
                                                      int nwg)
{
    constexpr int NS = ND - 1;  // at most this many distinct source patches
    constexpr int kNW = NT / 64;
    static_assert(NT >= 64 + ND, "threads 64 .. 64 + ND hold the direction keys");
    __shared__ int s_end[32];  // arrivals of the first 1, 2, ... sources; past the last source all of them
    __shared__ int64_t s_sbase[NS];
    __shared__ int s_key[ND];
    __shared__ int s_wc[kNW];
    __shared__ int s_run;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));

    for (int gp = wg; gp < total; gp += nwg) {
        const int s = find_sim(patch_prefix, nsims, gp);
        const SimDev<T> &S = sims[s];
        const int q = gp - patch_prefix[s];
        // everything that depends on q alone, loaded together: the state,
        // the patch's counts, and per thread one entry of its neighbour row
        // (threads below NS: a source and its key; threads 64 .. 64 + ND: a
        // direction's key)
        const uint32_t active = glb(S.st)->active, flags = glb(S.st)->flags;
        const int n = glb(S.count)[q], np = glb(S.newcount)[q], nH = glb(S.nhole)[q], A = glb(S.narrive)[q];
        const int L = glb(S.nleave)[q], nstaged = glb(S.kofs)[q * (ND + 1) + ND];
        const int64_t base = glb(S.off)[q];
        const gptr_t<const int32_t> row = nb_row<ND>(S.nbt, q);
        int r_ns = 0, r_a = 0, r_b = 0;
        if (tid < NS) {
            r_ns = row[ND];
            r_a = row[ND + 1 + tid];
            r_b = row[2 * ND + tid];
        } else if (tid >= 64 && tid < 64 + ND) {
            r_a = row[tid - 64];
        }
        if (!active || (flags & kFlagPending)) continue;
        if (A == 0 && np == n && L == 0) {
            // nothing arrives and nothing leaves
            if (tid == 0) {
                if (q == 0) glb(S.st)->rebinned = 1u;
                *glb(S.moved + q) = 0;
            }
            continue;
        }
        if (wave == 0) {
            // one lane per source: its count and staging base for this patch
            int end = 0;
            if (tid < NS && tid < r_ns) {
                const int sp = r_a, k = r_b;
                end = glb(S.kcnt)[sp * ND + k];
                s_sbase[tid] = glb(S.off)[sp] + glb(S.kofs)[sp * (ND + 1) + k];
            }
#pragma unroll
            for (int o = 1; o < 32; o <<= 1) {
                const int y = __shfl_up(end, o, 64);
                if (lane >= o) end += y;
            }
            if (lane < 32) s_end[lane] = end;
            if (tid == 0) {
                s_run = 0;
                if (q == 0) glb(S.st)->rebinned = 1u;
            }
        } else if (tid < 64 + ND) {
            s_key[tid - 64] = r_a;
        }
        __syncthreads();
        // arrivals (sources in ascending id, each in its slot order): holes
        // first, then appended from slot n; one thread per arrival, so the
        // copies of all sources are in flight together (its source from prefix
        // sums, not by a walk: 64 x 48 x 40 box 155 -> 152 us per step)
        for (int a = tid; a < A; a += NT) {
            int i = 0;  // the first source whose arrivals end after a
#pragma unroll
            for (int o = NS > 8 ? 16 : 4; o > 0; o >>= 1) i += a >= s_end[i + o - 1] ? o : 0;
            const int a0 = i ? s_end[i - 1] : 0;
            const int target = a < nH ? glb(S.holes)[base + a] : n + (a - nH);
            copy_particle(S, s_sbase[i] + (a - a0), base + target, true, false);
        }
        // stayers in [n', n) fill the remaining holes
        if (np < n) {
            for (int c0 = np; c0 < n; c0 += NT) {
                const int k = c0 + tid;
                bool stay = false;
                if (k < n) {
                    const uint8_t c = glb(S.code)[base + k];
                    stay = c != kRemoved && s_key[c] < 0;
                }
                const uint64_t b = __ballot(stay);
                if (lane == 0) s_wc[wave] = __popcll(b);
                __syncthreads();
                if (stay) {
                    int r = s_run + __popcll(b & lt);
                    for (int w = 0; w < wave; ++w) r += s_wc[w];
                    copy_particle(S, base + k, base + glb(S.holes)[base + A + r], false, false);
                }
                __syncthreads();
                if (tid == 0) {
                    int add = 0;
                    for (int w = 0; w < kNW; ++w) add += s_wc[w];
                    s_run += add;
                }
                __syncthreads();
            }
        }
        if (tid == 0) {
            glb(S.count)[q] = np;
            *glb(S.moved + q) = 0;
            const int removed = L - nstaged;
            if (removed)
                __hip_atomic_fetch_add(&glb(S.st)->removed, (uint64_t)removed, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
    }
}

}  // namespace pic
