// k winners-take-all with feature-wise and lateral inhibition (gfx950).
//
// Paper: section "snn Module" (winners chosen first by the earliest spike,
// then by the largest potential; lateral inhibition of the winner's
// surroundings in all feature maps) and "functional Module" (get_k_winners
// returning (feature, row, column) triplets; here with the spike step t).
//
// Every spiking neuron gets a unique 64-bit key whose unsigned order is the
// winner order:
//     bits 63..56  255 - t_first          (earlier spike wins)
//     bits 55..24  v_first, order-mapped  (larger potential wins)
//     bits 23..0   2^24 - 1 - index       (lower linear index wins ties)
// Silent neurons get key 0.  Two paths, by size:
//   * k <= 16 with per-position lists that fit in LDS: the k best keys of every
//     position, then k rounds without global reads ("per-position top-k");
//   * else the best key of every (run of feature maps, run of positions), found
//     again only where it was inhibited and could still win ("units").
#include <algorithm>

#include "common.hpp"

namespace {

__device__ __forceinline__ uint64_t kwta_key(int t, float v, uint32_t idx) {
    uint32_t u = __float_as_uint(v);
    u = u == 0x80000000u ? 0u : u;                        // -0 and +0 are equal potentials
    u ^= (uint32_t)((int32_t)u >> 31) | 0x80000000u;     // order-preserving: ~u if negative, else u | sign
    const uint32_t hi = ((uint32_t)(255 - t) << 24) | (u >> 8);
    const uint32_t lo = (u << 24) | (0xFFFFFFu - idx);
    return ((uint64_t)hi << 32) | lo;
}

// Maximum over the wave by DPP lane moves (the value of lane 63 after moves
// within quads, half-rows, rows, then across rows), returned to every lane.
// All 64 lanes must be active.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t max_dpp64(uint64_t v) {
    const int lo = (int)(uint32_t)v, hi = (int)(uint32_t)(v >> 32);
    const uint64_t o = ((uint64_t)(uint32_t)__builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xF, false) << 32) |
                       (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xF, false);
    return o > v ? o : v;
}
__device__ __forceinline__ uint64_t wave_max_u64_dpp(uint64_t v) {
    v = max_dpp64<0xB1, 0xF>(v);   // quad_perm [1,0,3,2]
    v = max_dpp64<0x4E, 0xF>(v);   // quad_perm [2,3,0,1]
    v = max_dpp64<0x141, 0xF>(v);  // row_half_mirror
    v = max_dpp64<0x140, 0xF>(v);  // row_mirror
    v = max_dpp64<0x142, 0xA>(v);  // row_bcast15 into rows 1, 3
    v = max_dpp64<0x143, 0xC>(v);  // row_bcast31 into rows 2, 3
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63);
    return ((uint64_t)hi << 32) | lo;
}

// n / d as umulhi(n, m) with m = ceil(2^32 / d); m == 0 stands for d == 1 (2^32 does not fit)
__device__ __forceinline__ unsigned qdiv(unsigned n, unsigned m) { return m ? __umulhi(n, m) : n; }

// ------------------------------------------------------------ per-position top-k
// When k <= 16 and each image's lists fit in LDS, one workgroup per image
// first keeps, for every position, the k largest keys over all feature maps:
// one pass over the image's neurons, with each position owned by one thread
// (on maps of few positions, the feature maps are split among up to
// TOPK_THREADS / HW threads per position, whose lists the owner then merges;
// small batches, which leave most CUs idle, take up to TOPK_THREADS_SMALL_B
// threads per workgroup so that each thread scans fewer feature maps).
// The rounds never read global memory again.  At round j at most j features
// are retired, so a position's best live key is among its first j + 1 list
// entries: the owner skips entries of retired features with a per-position
// cursor, and marks its position inhibited when it falls in a winner's
// window (with at most 4 positions per thread, the cursors and the current
// best keys live in registers).  Only the per-round maximum crosses threads.
constexpr int TOPK_THREADS = 256;       // most threads per workgroup
constexpr int TOPK_THREADS_SMALL_B = 1024;  // most threads per workgroup for batches below TOPK_SMALL_B
constexpr int TOPK_SMALL_B = 256;
constexpr int TOPK_MAX_K = 16;
constexpr size_t TOPK_LDS = 40 * 1024;  // lists and cursors (the stash adds 16 KB)
constexpr int TOPK_U = 8;               // feature maps loaded per block
constexpr int TOPK_STASH_MIN = 64;      // features per split from which the stash pays
constexpr int TOPK_RP = 4;              // positions per thread up to which the rounds keep their keys in registers
// Batches below TOPK_PRE_B images (online steps) leave most CUs idle: the
// lists are then built by a grid of (image, split of the feature maps)
// workgroups into the workspace, and the rounds' workgroup merges them.
constexpr int TOPK_PRE_B = 8;
constexpr int TOPK_PRE_NS = 16;         // feature splits at most
constexpr int TOPK_PRE_HW = 4096;       // positions at most

struct KwtaTopk {
    int B, T, C, HW, W, k, r;
    int S, fps;  // feature splits per position (small maps) and features per split
    int nt;      // threads per workgroup
    unsigned mHW, mW;
    int ns, fps2;  // workgroup feature splits and their features (ns > 1: lists built by k_kwta_lists)
    uint64_t *lg;  // their lists, [B][ns][HW][KM]
};

// Inserts key into the descending list top (keys are unique; the caller has
// checked key > top[KM - 1], so the last entry drops out).
template <int KM>
__device__ __forceinline__ void topk_insert(uint64_t (&top)[KM], uint64_t key) {
    bool gt[KM];  // every comparison first, then the moves
#pragma unroll
    for (int i = 0; i < KM; ++i) gt[i] = key > top[i];
#pragma unroll
    for (int i = KM - 1; i > 0; --i) top[i] = gt[i - 1] ? top[i - 1] : (gt[i] ? key : top[i]);
    top[0] = gt[0] ? key : top[0];
}

// Grid (image, split): the KM best keys of every position over the split's
// feature maps, into g.lg.
template <int KM, int U>
__global__ __launch_bounds__(TOPK_THREADS_SMALL_B) void k_kwta_lists(const uint8_t *__restrict__ tf_all,
                                                             const float *__restrict__ vf_all, KwtaTopk g) {
    const int b = blockIdx.x, sp = blockIdx.y, HW = g.HW;
    const int64_t N = (int64_t)g.C * HW;
    const uint8_t *tf = tf_all + (int64_t)b * N;
    const float *vf = vf_all + (int64_t)b * N;
    const int fa = sp * g.fps2, fb = min(g.C, fa + g.fps2);
    for (int p = threadIdx.x; p < HW; p += blockDim.x) {
        uint64_t top[KM];
#pragma unroll
        for (int i = 0; i < KM; ++i) top[i] = 0;
        for (int f0 = fa; f0 < fb; f0 += U) {
            int tv[U];
            float vv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool ok = f0 + u < fb;
                const int o = (f0 + u) * HW + p;
                tv[u] = ok ? (int)tf[o] : g.T;
                vv[u] = ok ? vf[o] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (tv[u] < g.T) {
                    const uint64_t key = kwta_key(tv[u], vv[u], (uint32_t)((f0 + u) * HW + p));
                    if (key > top[KM - 1]) topk_insert(top, key);
                }
            }
        }
        uint64_t *dst = g.lg + (((int64_t)b * g.ns + sp) * HW + p) * KM;
#pragma unroll
        for (int i = 0; i < KM; ++i) dst[i] = top[i];
    }
}

template <int KM, int U, bool STASH>
__global__ __launch_bounds__(TOPK_THREADS_SMALL_B) void k_kwta_topk(const uint8_t *__restrict__ tf_all,
                                                            const float *__restrict__ vf_all, KwtaTopk g,
                                                            int32_t *__restrict__ winners,
                                                            int32_t *__restrict__ n_winners) {
    extern __shared__ uint64_t lists[];  // [S][HW][KM] keys, then [HW] cursors
    uint8_t *cur = reinterpret_cast<uint8_t *>(lists + (size_t)g.S * g.HW * KM);
    __shared__ uint64_t red[2][TOPK_THREADS_SMALL_B / 64];
    // a block's keys, read back by their own lane (STASH launches have at most TOPK_THREADS threads)
    __shared__ uint64_t stash[STASH ? U : 1][TOPK_THREADS];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int NT = blockDim.x, NW = NT >> 6;
    const int HW = g.HW, S = g.S;
    const int64_t N = (int64_t)g.C * HW;
    const uint8_t *tf = tf_all + (int64_t)b * N;
    const float *vf = vf_all + (int64_t)b * N;
    int32_t *win = winners + (int64_t)b * g.k * 4;
    for (int i = tid; i < 4 * g.k; i += NT) win[i] = -1;

    // The lists of the workgroup splits, merged (each is sorted), MB of them read whole
    // before the first is merged: an entry at a time, each waited for, one image of 250
    // maps of 14x14, k = 8, took 24.7 us, now 22.2.  (Several threads per position, their
    // lists merged again by the owner: 29 us.)
    for (int p = tid; p < (g.ns > 1 ? HW : 0); p += NT) {
        constexpr int MB = KM <= 8 ? 4 : KM <= 12 ? 2 : 1;
        uint64_t top[KM];
#pragma unroll
        for (int i = 0; i < KM; ++i) top[i] = 0;
        for (int sp0 = 0; sp0 < g.ns; sp0 += MB) {
            uint64_t kk[MB][KM];
#pragma unroll
            for (int q = 0; q < MB; ++q) {
                const uint64_t *src = g.lg + (((int64_t)b * g.ns + min(sp0 + q, g.ns - 1)) * HW + p) * KM;
#pragma unroll
                for (int e = 0; e < KM; ++e) kk[q][e] = src[e];
            }
#pragma unroll
            for (int q = 0; q < MB; ++q) {
                if (sp0 + q >= g.ns) break;
#pragma unroll
                for (int e = 0; e < KM; ++e) {
                    if (!(kk[q][e] > top[KM - 1])) break;
                    topk_insert(top, kk[q][e]);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < KM; ++i) lists[(size_t)p * KM + i] = top[i];
    }
    // pass over the image: the KM best keys of every (position, feature split)
    for (int pp = tid; pp < (g.ns > 1 ? 0 : HW * S); pp += NT) {
        const int s = (int)qdiv((unsigned)pp, g.mHW), p = pp - s * HW;
        uint64_t top[KM];
#pragma unroll
        for (int i = 0; i < KM; ++i) top[i] = 0;
        const int fa = s * g.fps, fb = min(g.C, fa + g.fps);
        for (int f0 = fa; f0 < fb; f0 += U) {
            int tv[U];
            float vv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool ok = f0 + u < fb;
                const int o = (f0 + u) * HW + p;
                tv[u] = ok ? (int)tf[o] : g.T;
                vv[u] = ok ? vf[o] : 0.0f;
            }
            if constexpr (STASH) {
                // the keys that beat the list's last entry are inserted after the
                // block, each lane walking only its own: the wave then loops as
                // often as its busiest lane rather than once per key any lane keeps
                unsigned pass = 0;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint64_t key = tv[u] < g.T ? kwta_key(tv[u], vv[u], (uint32_t)((f0 + u) * HW + p)) : 0;
                    stash[u][tid] = key;
                    pass |= (key > top[KM - 1] ? 1u : 0u) << u;
                }
                while (pass) {
                    const int j = __builtin_ctz(pass);
                    pass &= pass - 1;
                    const uint64_t key = stash[j][tid];
                    if (key > top[KM - 1]) topk_insert(top, key);
                }
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (tv[u] < g.T) {
                        const uint64_t key = kwta_key(tv[u], vv[u], (uint32_t)((f0 + u) * HW + p));
                        if (key > top[KM - 1]) topk_insert(top, key);
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < KM; ++i) lists[(size_t)pp * KM + i] = top[i];
    }
    if (S > 1 && g.ns <= 1) {  // uniform
        __syncthreads();
        // owners fold the other splits' lists into their own
        for (int p = tid; p < HW; p += NT) {
            uint64_t top[KM];
#pragma unroll
            for (int i = 0; i < KM; ++i) top[i] = lists[(size_t)p * KM + i];
            for (int s = 1; s < S; ++s)
                for (int e = 0; e < KM; ++e) {
                    const uint64_t key = lists[((size_t)s * HW + p) * KM + e];
                    if (!(key > top[KM - 1])) break;  // the split's list is sorted
                    topk_insert(top, key);
                }
#pragma unroll
            for (int i = 0; i < KM; ++i) lists[(size_t)p * KM + i] = top[i];
        }
    }
    int deadf[KM];
#pragma unroll
    for (int j = 0; j < KM; ++j) deadf[j] = -1;
    int found = 0;
    auto feature = [&](uint64_t key) { return (int)qdiv(0xFFFFFFu - (unsigned)(key & 0xFFFFFFu), g.mHW); };
    auto is_dead = [&](int f) {
        bool dead = false;
#pragma unroll
        for (int j = 0; j < KM; ++j) dead |= deadf[j] == f;
        return dead;
    };
    if (HW <= TOPK_RP * NT) {  // uniform
        // Each thread holds the best live key of each of its positions in
        // registers (0: none, or inhibited).  A round changes it only where the
        // winner's window covers the position, or where the cached key belongs to
        // the winner's feature: then the list is walked on to the next entry of a
        // live feature (the cached key stays the best live one otherwise).
        uint64_t bk[TOPK_RP];
        int cc[TOPK_RP], py[TOPK_RP], px[TOPK_RP];
#pragma unroll
        for (int i = 0; i < TOPK_RP; ++i) {
            const int p = tid + i * NT;
            bk[i] = p < HW ? lists[(size_t)p * KM] : 0;
            cc[i] = 0;
            py[i] = (int)qdiv((unsigned)min(p, HW - 1), g.mW);
            px[i] = min(p, HW - 1) - py[i] * g.W;
        }
        for (int round = 0; round < g.k; ++round) {
            uint64_t m = 0;
#pragma unroll
            for (int i = 0; i < TOPK_RP; ++i) m = bk[i] > m ? bk[i] : m;
            m = wave_max_u64_dpp(m);
            if (lane == 0) red[round & 1][wv] = m;
            __syncthreads();
            uint64_t best = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) best = red[round & 1][w] > best ? red[round & 1][w] : best;
            if (best == 0) break;  // uniform
            const int idx = (int)(0xFFFFFFu - (unsigned)(best & 0xFFFFFFu));
            const int t = 255 - (int)(best >> 56);
            const int fw = (int)qdiv((unsigned)idx, g.mHW);
            const int pos = idx - fw * HW;
            const int yw = (int)qdiv((unsigned)pos, g.mW);
            const int xw = pos - yw * g.W;
            if (tid == 0) {
                win[4 * round + 0] = fw;
                win[4 * round + 1] = t;
                win[4 * round + 2] = yw;
                win[4 * round + 3] = xw;
            }
#pragma unroll
            for (int j = 0; j < KM; ++j)
                if (j == found) deadf[j] = fw;
            ++found;
#pragma unroll
            for (int i = 0; i < TOPK_RP; ++i) {
                if (bk[i] == 0) continue;
                if (abs(py[i] - yw) <= g.r && abs(px[i] - xw) <= g.r) {
                    bk[i] = 0;
                    continue;
                }
                if (feature(bk[i]) != fw) continue;
                const int p = tid + i * NT;
                uint64_t key = 0;
                for (int c = cc[i] + 1; c < KM; ++c) {
                    const uint64_t e = lists[(size_t)p * KM + c];
                    if (e == 0) break;
                    if (!is_dead(feature(e))) {
                        key = e;
                        cc[i] = c;
                        break;
                    }
                }
                bk[i] = key;
            }
        }
    } else {
        for (int p = tid; p < HW; p += NT) cur[p] = 0;
        for (int round = 0; round < g.k; ++round) {
            uint64_t m = 0;
            for (int p = tid; p < HW; p += NT) {
                int c = cur[p];
                if (c == 0xFF) continue;  // laterally inhibited
                const int c0 = c;
                uint64_t key = 0;
                for (; c < KM; ++c) {
                    key = lists[(size_t)p * KM + c];
                    if (key == 0) break;
                    if (!is_dead(feature(key))) break;
                    key = 0;
                }
                if (c != c0) cur[p] = (uint8_t)c;
                m = key > m ? key : m;
            }
            m = wave_max_u64_dpp(m);
            if (lane == 0) red[round & 1][wv] = m;
            __syncthreads();
            uint64_t best = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) best = red[round & 1][w] > best ? red[round & 1][w] : best;
            if (best == 0) break;  // uniform
            const int idx = (int)(0xFFFFFFu - (unsigned)(best & 0xFFFFFFu));
            const int t = 255 - (int)(best >> 56);
            const int fw = (int)qdiv((unsigned)idx, g.mHW);
            const int pos = idx - fw * HW;
            const int yw = (int)qdiv((unsigned)pos, g.mW);
            const int xw = pos - yw * g.W;
            if (tid == 0) {
                win[4 * round + 0] = fw;
                win[4 * round + 1] = t;
                win[4 * round + 2] = yw;
                win[4 * round + 3] = xw;
            }
#pragma unroll
            for (int j = 0; j < KM; ++j)
                if (j == found) deadf[j] = fw;
            ++found;
            for (int p = tid; p < HW; p += NT) {
                const int y = (int)qdiv((unsigned)p, g.mW), x = p - y * g.W;
                if (abs(y - yw) <= g.r && abs(x - xw) <= g.r) cur[p] = 0xFF;
            }
        }
    }
    if (tid == 0) n_winners[b] = found;
}

// ------------------------------------------------------------ units
// A unit is a run of feature maps times a run of 64 * L consecutive positions,
// the work of one wave.  k_kwta_units writes every unit's best key; the rounds
// (k_kwta_rounds, one workgroup per image) hold the keys in registers.  A key
// whose feature was retired or whose position was inhibited since is an upper
// bound of its unit; only the units whose bound exceeds the best valid key are
// read again, each by its wave.
// Why units and not the maxima of single feature maps: features that see the
// same input have their maxima at the same places, so one winner inhibits the
// maximum of every map; with runs of maps it inhibits those of the runs at its
// place only.  Runs of all maps would suffer in the opposite case, a feature
// that is the best almost everywhere.  Hence runs of UN_MAPS maps, which one wave
// reads at once, longer where that makes more than UN_MAX units: 256 maps of
// 256x256 make 256 x 16 units of 256 positions x 16 maps, 20 KB to read again; 250
// of 14x14 make 4 x 32 units of 64 positions x 8 maps.
// Bound by the one pass over the maps (5 bytes a neuron) and k rounds of two
// reductions each.  With the maxima of tiles of 16 rows, all of them read again
// whose maximum was inhibited, 4 images of 256 maps of 256x256, k = 32, took
// 14.6 ms; now 0.48 ms, 79 us of it the pass (4.3 TB/s) and the rest the
// latency of the rounds' reads (5 to 14 us a round).  Smaller maps whose features
// spike at the same places, k = 32, 32 images: 250 of 14x14 176 us with the maxima
// of tiles, 429 with runs of one map, 163 so; 256 of 64x64 1770, 2540 and 592 (runs
// of 4 maps 1013, of 16 698).
constexpr int UN_MAX = 4096;      // units per image at most (8 bytes each in the workspace)
constexpr int UN_UPT = 4;         // units per thread of the rounds
constexpr int UN_THREADS = UN_MAX / UN_UPT;
// Few waves wait longer for what a round reads again, many for each other at its
// barriers (250 maps of 14x14, one image, k = 32, shared places: 4 waves 267 us, 8 167,
// 16 162; independent ones 99, 78, 97).
constexpr int UN_MIN_THREADS = 512;
// Units of 64 positions up to here, of 256 beyond: narrow ones are less to read again, but
// more to hold (32 images, k = 32, shared places, 64 : 256 positions: 30 maps of 64x64 118 :
// 154 us, 20 of 90x90 84 : 102).
constexpr int UN_NARROW = 1024;
constexpr int UN_MAPS = 8;        // maps a wave reads at once
constexpr int UN_MAX_C = 4096;    // feature maps at most (the retired ones' bitmap)

struct KwtaUnits {
    int B, T, C, HW, W, k, r;
    int L;              // positions per lane: 1 or 4
    int ns, fps;        // runs of feature maps and maps per run
    int groups, units;  // runs of 64 * L positions, ns * groups
    int vec;            // L == 4 with aligned 4-byte / 16-byte loads
    unsigned mHW;       // ceil(2^32 / HW) (0 for 1)
    uint64_t *ukey;     // [B][units], unit = group * ns + run
};

// The feature of a key: the estimated quotient is exact or one too large.
__device__ __forceinline__ int unit_feature(const KwtaUnits &g, uint64_t key, int &pos) {
    const unsigned idx = 0xFFFFFFu - (unsigned)(key & 0xFFFFFFu);
    int f = (int)qdiv(idx, g.mHW);
    pos = (int)idx - f * g.HW;
    if (pos < 0) {
        --f;
        pos += g.HW;
    }
    return f;
}

// The best key of unit u's feature maps fa..fb-1 over the live features and
// positions, by one wave (bitmaps of the retired features and inhibited
// positions, or null).
template <int L>
__device__ __forceinline__ uint64_t unit_best(const uint8_t *__restrict__ tf, const float *__restrict__ vf,
                                              const KwtaUnits &g, int grp, int fa, int fb, int lane,
                                              const uint32_t *dead, const uint32_t *inh) {
    constexpr int U = UN_MAPS;
    const int p = (grp * 64 + lane) * L;
    unsigned ok = 0;  // positions that count
#pragma unroll
    for (int j = 0; j < L; ++j) ok |= (p + j < g.HW ? 1u : 0u) << j;
    if (inh && ok) ok &= ~(inh[p >> 5] >> (p & 31));
    uint64_t m = 0;
    for (int f0 = fa; f0 < fb; f0 += U) {
        // the block's live maps (uniform), then the last of them again in place of the others
        uint32_t live = (1u << min(U, fb - f0)) - 1u;
        if (dead) {
            const uint64_t d = (uint64_t)dead[(f0 >> 5) + 1] << 32 | dead[f0 >> 5];
            live &= ~(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(d >> (f0 & 31)));
        }
        if (live == 0) continue;
        int fq[U];
        const int n = __popc(live);
#pragma unroll
        for (int q = 0; q < U; ++q) {
            fq[q] = f0 + __ffs((int)live) - 1;
            live = live & (live - 1) ? live & (live - 1) : live;
        }
        uint32_t tw[U];  // L first-spike times, a byte each
        float vv[U][L];
#pragma unroll
        for (int q = 0; q < U; ++q) {  // (unconditional loads, all in flight)
            const int o = fq[q] * g.HW;
            if (L == 4 && g.vec) {     // (whole quads: HW is a multiple of 4)
                const int oq = o + min(p, g.HW - 4);
                tw[q] = *reinterpret_cast<const uint32_t *>(tf + oq);
                const float4 x = *reinterpret_cast<const float4 *>(vf + oq);
                vv[q][0] = x.x;
                vv[q][L > 1 ? 1 : 0] = L > 1 ? x.y : x.x;
                vv[q][L > 2 ? 2 : 0] = L > 2 ? x.z : x.x;
                vv[q][L > 3 ? 3 : 0] = L > 3 ? x.w : x.x;
            } else {
                tw[q] = 0;
#pragma unroll
                for (int j = 0; j < L; ++j) {
                    const int oj = o + min(p + j, g.HW - 1);
                    tw[q] |= (uint32_t)tf[oj] << (8 * j);
                    vv[q][j] = vf[oj];
                }
            }
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int f = fq[q];
            if (q >= n) continue;  // uniform
#pragma unroll
            for (int j = 0; j < L; ++j) {
                const int t = (int)((tw[q] >> (8 * j)) & 255u);
                if (((ok >> j) & 1u) && t < g.T) {
                    const uint64_t key = kwta_key(t, vv[q][j], (uint32_t)(f * g.HW + p + j));
                    m = key > m ? key : m;
                }
            }
        }
    }
    return wave_max_u64_dpp(m);
}

// Grid: image (from b0 on) * ceil(units / 4) blocks of 4 units, one wave each.
// Consecutive units are the runs of maps at one place.
__global__ __launch_bounds__(256) void k_kwta_units(const uint8_t *__restrict__ tf, const float *__restrict__ vf,
                                                    KwtaUnits g, int b0) {
    const int nblk = (g.units + 3) / 4, lane = threadIdx.x & 63, bi = blockIdx.x / nblk;
    const int b = b0 + bi, u = (int)(blockIdx.x - bi * nblk) * 4 + (int)(threadIdx.x >> 6);
    if (u >= g.units) return;
    const int64_t N = (int64_t)g.C * g.HW;
    const int grp = u / g.ns, fa = (u - grp * g.ns) * g.fps, fb = min(g.C, fa + g.fps);
    const uint64_t m = g.L == 4 ? unit_best<4>(tf + b * N, vf + b * N, g, grp, fa, fb, lane, nullptr, nullptr)
                                : unit_best<1>(tf + b * N, vf + b * N, g, grp, fa, fb, lane, nullptr, nullptr);
    if (lane == 0) g.ukey[(int64_t)b * g.units + u] = m;
}

template <int L>
__global__ __launch_bounds__(UN_THREADS) void k_kwta_rounds(const uint8_t *__restrict__ tf_all,
                                                            const float *__restrict__ vf_all, KwtaUnits g, int b0,
                                                            int32_t *__restrict__ winners,
                                                            int32_t *__restrict__ n_winners) {
    extern __shared__ uint32_t inh[];         // bitmap of the inhibited positions
    __shared__ uint32_t dead[UN_MAX_C / 32 + 1];  // bitmap of the retired features
    __shared__ uint64_t red[2][UN_THREADS / 64];
    __shared__ uint64_t res[UN_MAX];          // the listed units' new keys
    __shared__ uint16_t list[UN_MAX];
    __shared__ int nlist;
    const int b = b0 + (int)blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int NT = blockDim.x, NW = NT >> 6, nwords = (g.HW + 31) / 32;
    const int64_t N = (int64_t)g.C * g.HW;
    const uint8_t *tf = tf_all + b * N;
    const float *vf = vf_all + b * N;
    int32_t *win = winners + (int64_t)b * g.k * 4;
    for (int i = tid; i < nwords; i += NT) inh[i] = 0;
    for (int i = tid; i < UN_MAX_C / 32 + 1; i += NT) dead[i] = 0;
    for (int i = tid; i < 4 * g.k; i += NT) win[i] = -1;
    uint64_t K[UN_UPT];
#pragma unroll
    for (int i = 0; i < UN_UPT; ++i) {
        const int u = i * NT + tid;
        K[i] = u < g.units ? g.ukey[(int64_t)b * g.units + u] : 0;
    }
    const int nsub = (g.fps + UN_MAPS - 1) / UN_MAPS;  // parts of a unit's maps, a wave each
    if (tid == 0) nlist = 0;
    __syncthreads();
    int found = 0;
    const int rounds = min(g.k, g.C);  // (each retires a feature)
    for (int round = 0; round < rounds; ++round) {
        bool valid[UN_UPT];
        uint64_t m = 0;
#pragma unroll
        for (int i = 0; i < UN_UPT; ++i) {
            int pos;
            const int f = unit_feature(g, K[i], pos);
            valid[i] = K[i] != 0 && !((dead[f >> 5] >> (f & 31)) & 1u) && !((inh[pos >> 5] >> (pos & 31)) & 1u);
            m = valid[i] && K[i] > m ? K[i] : m;
        }
        m = wave_max_u64_dpp(m);
        if (lane == 0) red[0][wv] = m;
        __syncthreads();
        uint64_t best = 0;
        for (int w = 0; w < NW; ++w) best = red[0][w] > best ? red[0][w] : best;
        // the units to read again, then their maps in parts dealt out to the waves
        int at[UN_UPT];
#pragma unroll
        for (int i = 0; i < UN_UPT; ++i) {
            at[i] = -1;
            if (!valid[i] && K[i] > best) {
                at[i] = atomicAdd(&nlist, 1);
                list[at[i]] = (uint16_t)(i * NT + tid);
                res[at[i]] = 0;
            }
        }
        __syncthreads();
        const int nl = nlist;
        for (int e = wv; e < nl * nsub; e += NW) {
            const int li = e / nsub, u = list[li], grp = u / g.ns, sp = u - grp * g.ns;
            const int fa = sp * g.fps + (e - li * nsub) * UN_MAPS, fb = min(min(g.C, (sp + 1) * g.fps), fa + UN_MAPS);
            if (fa >= fb) continue;  // (the last run's maps may be fewer)
            const uint64_t key = unit_best<L>(tf, vf, g, grp, fa, fb, lane, dead, inh);
            if (lane == 0 && key) atomicMax(reinterpret_cast<unsigned long long *>(&res[li]), (unsigned long long)key);
        }
        __syncthreads();
        m = 0;
#pragma unroll
        for (int i = 0; i < UN_UPT; ++i)
            if (at[i] >= 0) {
                K[i] = res[at[i]];
                m = K[i] > m ? K[i] : m;
            }
        m = wave_max_u64_dpp(m);
        if (lane == 0) red[1][wv] = m;
        if (tid == 0) nlist = 0;
        __syncthreads();
        for (int w = 0; w < NW; ++w) best = red[1][w] > best ? red[1][w] : best;
        if (best == 0) break;  // uniform: every thread read the same red[]
        int pos;
        const int fw = unit_feature(g, best, pos);
        const int yw = pos / g.W, xw = pos - yw * g.W, H = g.HW / g.W;
        if (tid == 0) {
            win[4 * round + 0] = fw;
            win[4 * round + 1] = 255 - (int)(best >> 56);
            win[4 * round + 2] = yw;
            win[4 * round + 3] = xw;
            dead[fw >> 5] |= 1u << (fw & 31);
        }
        ++found;
        const int ya = max(0, yw - min(g.r, yw)), yb = min(H - 1, yw + min(g.r, H));
        const int xa = max(0, xw - min(g.r, xw)), xb = min(g.W - 1, xw + min(g.r, g.W));
        const int ww = xb - xa + 1, wh = yb - ya + 1;
        for (int i = tid; i < wh * ww; i += NT) {
            const int q = (ya + i / ww) * g.W + xa + i % ww;
            atomicOr(&inh[q >> 5], 1u << (q & 31));
        }
        __syncthreads();
    }
    if (tid == 0) n_winners[b] = found;
}

KwtaUnits kwta_units(int B, int T, int C, int H, int W, int k, int r) {
    KwtaUnits g{};
    g.B = B; g.T = T; g.C = C; g.HW = H * W; g.W = W; g.k = k; g.r = r;
    g.L = (g.HW + 63) / 64 * ((C + UN_MAPS - 1) / UN_MAPS) > UN_NARROW ? 4 : 1;
    g.groups = (int)spk::ceil_div(g.HW, 64 * g.L);  // at most 256
    const int ns = std::min((C + UN_MAPS - 1) / UN_MAPS, UN_MAX / g.groups);
    g.fps = (C + ns - 1) / ns;
    g.ns = (C + g.fps - 1) / g.fps;
    g.units = g.ns * g.groups;
    g.mHW = g.HW == 1 ? 0u : (unsigned)(((1ULL << 32) + (uint64_t)g.HW - 1) / (uint64_t)g.HW);
    return g;
}

bool kwta_topk(int B, int T, int C, int H, int W, int k, int r, KwtaTopk &s) {
    const int64_t HW = (int64_t)H * W;
    if (k > TOPK_MAX_K || HW > 65536) return false;
    // maps of few positions split the feature maps among up to NT / HW threads per position
    const int NT = B < TOPK_SMALL_B ? TOPK_THREADS_SMALL_B : TOPK_THREADS;
    int S = HW <= NT ? (int)std::min<int64_t>(C, NT / HW) : 1;
    while (S > 1 && (size_t)HW * (S * k * sizeof(uint64_t) + 1) > TOPK_LDS) --S;  // the splits' lists fit
    const int fps = (C + S - 1) / S;
    S = (C + fps - 1) / fps;
    // threads: whole waves covering HW * S in as few passes as NT allows
    const int64_t work = HW * S, passes = (work + NT - 1) / NT;
    const int nt = (int)(((work + passes - 1) / passes + 63) / 64 * 64);
    if ((size_t)HW * (S * k * sizeof(uint64_t) + 1) > TOPK_LDS) return false;
    auto magic = [](int64_t d) {  // 0 for d == 1 (see qdiv)
        return d == 1 ? 0u : (unsigned)(((1ULL << 32) + (uint64_t)d - 1) / (uint64_t)d);
    };
    auto exact = [](int64_t d, int64_t n) {  // umulhi(x, ceil(2^32/d)) == x/d for all x < n
        const uint64_t m = ((1ULL << 32) + (uint64_t)d - 1) / (uint64_t)d;
        const uint64_t e = m * (uint64_t)d - (1ULL << 32);
        return (uint64_t)n * e < (1ULL << 32);
    };
    if (!exact(HW, (int64_t)C * HW) || !exact(W, HW)) return false;
    s = KwtaTopk{B, T, C, (int)HW, W, k, r, S, fps, nt, magic(HW), magic(W), 1, C, nullptr};
    if (B < TOPK_PRE_B && HW <= TOPK_PRE_HW) {  // lists by a grid of workgroups (the rounds' workgroup: S = 1)
        const int ns = (int)std::min<int64_t>(TOPK_PRE_NS, (C + 15) / 16);
        if (ns > 1) {
            s.ns = ns;
            s.fps2 = (C + ns - 1) / ns;
            s.ns = (C + s.fps2 - 1) / s.fps2;
            s.S = 1;
            s.fps = C;
            const int64_t passes = (HW + NT - 1) / NT;
            s.nt = (int)(((HW + passes - 1) / passes + 63) / 64 * 64);
        }
    }
    return true;
}

template <int KM>
void launch_topk(const KwtaTopk &s, const uint8_t *tf, const float *vf, int32_t *winners, int32_t *nw,
                 hipStream_t st) {
    const size_t lds = (size_t)s.HW * (s.S * KM * sizeof(uint64_t) + 1);
    if (s.ns > 1) {
        const int nt = (int)std::min<int64_t>(TOPK_THREADS_SMALL_B, ((int64_t)s.HW + 63) / 64 * 64);
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_kwta_lists<KM, TOPK_U>), dim3(s.B, s.ns), dim3(nt), 0, st, tf, vf, s);
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_kwta_topk<KM, TOPK_U, false>), dim3(s.B), dim3(s.nt), lds, st, tf, vf,
                           s, winners, nw);
        return;
    }
    if (s.fps >= TOPK_STASH_MIN && s.nt <= TOPK_THREADS)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_kwta_topk<KM, TOPK_U, true>), dim3(s.B), dim3(s.nt), lds, st, tf, vf, s,
                           winners, nw);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_kwta_topk<KM, TOPK_U, false>), dim3(s.B), dim3(s.nt), lds, st, tf, vf, s,
                           winners, nw);
}

void dispatch_topk(const KwtaTopk &s, const uint8_t *tf, const float *vf, int32_t *winners, int32_t *nw,
                   hipStream_t st) {
    switch (s.k) {
#define SPK_TOPK(K) \
    case K: launch_topk<K>(s, tf, vf, winners, nw, st); break;
        SPK_TOPK(1) SPK_TOPK(2) SPK_TOPK(3) SPK_TOPK(4) SPK_TOPK(5) SPK_TOPK(6) SPK_TOPK(7) SPK_TOPK(8)
        SPK_TOPK(9) SPK_TOPK(10) SPK_TOPK(11) SPK_TOPK(12) SPK_TOPK(13) SPK_TOPK(14) SPK_TOPK(15) SPK_TOPK(16)
#undef SPK_TOPK
        default: break;
    }
}

int kwta_check(int B, int T, int C, int H, int W, int k, int r) {
    SPK_REQUIRE(B >= 0 && T >= 1 && C >= 1 && H >= 1 && W >= 1, SPK_E_SHAPE, "spk_kwta: bad sizes");
    SPK_REQUIRE(T <= 255, SPK_E_RANGE, "spk_kwta: T=%d > 255", T);
    SPK_REQUIRE((int64_t)C * H * W <= (1LL << 24), SPK_E_RANGE, "spk_kwta: C*H*W > 2^24");
    SPK_REQUIRE((int64_t)H * W <= 65536, SPK_E_RANGE, "spk_kwta: H*W > 65536");
    SPK_REQUIRE(k >= 1 && r >= 0, SPK_E_ARG, "spk_kwta: k=%d must be >= 1 and radius=%d >= 0", k, r);
    SPK_REQUIRE(C <= UN_MAX_C, SPK_E_RANGE, "spk_kwta: %d feature maps exceed %d", C, UN_MAX_C);
    // The batch limit of the call, kept as it is whatever the kernels' launches need (they stay below
    // it): with maps cut into tiles of RB rows so that an image has at most UN_MAX, and G lanes, up to
    // 64, that cover a tile, fewer than 2^31 lanes in all.
    int RB = 1, G = 1;
    while (RB < H && (int64_t)C * ((H + RB - 1) / RB) > UN_MAX) RB *= 2;
    RB = std::min(RB, H);
    while (G < RB * W && G < 64) G <<= 1;
    SPK_REQUIRE((int64_t)B * C * ((H + RB - 1) / RB) * G < (1LL << 31), SPK_E_RANGE, "spk_kwta: batch too large");
    return SPK_OK;
}

}  // namespace

extern "C" size_t spk_kwta_workspace_size(int B, int C, int H, int W) {
    if (kwta_check(B, 1, C, H, W, 1, 0) != SPK_OK) return 0;
    const KwtaUnits u = kwta_units(B, 1, C, H, W, 1, 0);
    size_t need = (size_t)B * u.units * sizeof(uint64_t);
    if (B < TOPK_PRE_B && (int64_t)H * W <= TOPK_PRE_HW)  // the workgroup splits' lists (any k up to TOPK_MAX_K)
        need = std::max(need, (size_t)B * TOPK_PRE_NS * H * W * TOPK_MAX_K * sizeof(uint64_t));
    return spk::align_up(need, 256);
}

extern "C" int spk_kwta(const uint8_t *t_first, const float *v_first, int B, int T, int C, int H, int W, int k,
                        int radius, int32_t *winners, int32_t *n_winners, void *workspace, size_t ws_bytes,
                        void *stream) {
    int rc = kwta_check(B, T, C, H, W, k, radius);
    if (rc != SPK_OK) return rc;
    if (B == 0) return spk::ok();
    SPK_REQUIRE(t_first && v_first && winners && n_winners, SPK_E_ARG,
                "spk_kwta: t_first, v_first, winners and n_winners are required");
    const size_t need = spk_kwta_workspace_size(B, C, H, W);
    SPK_REQUIRE(workspace && ws_bytes >= need, SPK_E_WORKSPACE, "spk_kwta: workspace of %zu bytes < %zu required",
                ws_bytes, need);
    hipStream_t st = spk::as_stream(stream);
    KwtaTopk tk;
    if (kwta_topk(B, T, C, H, W, k, radius, tk)) {
        tk.lg = static_cast<uint64_t *>(workspace);
        dispatch_topk(tk, t_first, v_first, winners, n_winners, st);
        return spk::check_launch("spk_kwta");
    }
    KwtaUnits g = kwta_units(B, T, C, H, W, k, radius);
    g.ukey = static_cast<uint64_t *>(workspace);
    g.vec = g.L == 4 && g.HW % 4 == 0 && ((uintptr_t)t_first & 3) == 0 && ((uintptr_t)v_first & 15) == 0;
    const int nblk = (g.units + 3) / 4, most = ((1 << 24) - 1) / nblk;  // a launch has fewer than 2^32 threads
    for (int64_t b0 = 0; b0 < B; b0 += most)
        hipLaunchKernelGGL(k_kwta_units, dim3((unsigned)(std::min<int64_t>(most, B - b0) * nblk)), dim3(256), 0, st,
                           t_first, v_first, g, (int)b0);
    const int nt = (int)std::max<int64_t>(g.L == 1 && g.ns >= 24 ? UN_THREADS : UN_MIN_THREADS,
                                          spk::align_up((size_t)spk::ceil_div(g.units, UN_UPT), 64));
    const size_t lds = (size_t)(g.HW + 31) / 32 * 4;
    const int64_t imgs = ((1LL << 32) - 1) / nt;
    for (int64_t b0 = 0; b0 < B; b0 += imgs) {
        const dim3 grid((unsigned)std::min<int64_t>(imgs, B - b0));
        if (g.L == 4)
            hipLaunchKernelGGL(k_kwta_rounds<4>, grid, dim3(nt), lds, st, t_first, v_first, g, (int)b0, winners,
                               n_winners);
        else
            hipLaunchKernelGGL(k_kwta_rounds<1>, grid, dim3(nt), lds, st, t_first, v_first, g, (int)b0, winners,
                               n_winners);
    }
    return spk::check_launch("spk_kwta");
}
