// walk.hip -- persistent random-walk kernel in a homogeneous sphere
// (training-data process of Sec. 3.1; exit parameterisation of Sec. 4.1;
// representative event of Sec. 4.3).
//
// One photon per lane at a time.  Scattering-chain lengths are heavy tailed
// (1 to ~10^5 events), so lanes take new photons from a per-wave ticket pool
// as soon as theirs leaves the sphere: waves stay full until the global
// ticket counter runs past n_photons.  The rest of the run is the last long
// chains on nearly empty waves: training walks are handed out longest expected
// chain first (a counting sort of the photon ids by a bucket of sigma_t r and
// g), and a wave with few chains left walks them together.  Each photon's
// result depends only on its id, so neither changes an output.
#include "host.hpp"
#include "mfma.hpp"

namespace msst {

struct WalkArgs {
    uint64_t seed, photon_offset, n;
    float sigma_t, g, albedo, radius, r2, st_report;
    uint32_t surv_thr;  // survive iff u24 <= floor(albedo 2^24)
    float st_lo, st_log2_ratio, g_lo, g_span, a_lo, a_span;
    uint32_t focus_thr;  // focus iff u24 <= floor(focus_fraction 2^24); 0 = never
    float fst_lo, fst_log2_ratio, fg_lo, fg_span;
    int32_t weighting;
    uint32_t max_events;
    float* params;
    uint32_t* n_scatter;
    uint32_t* event_index;
    uint8_t* absorbed;
    uint8_t* truncated;
    float* exit_pos;
    float* exit_dir;
    float* exit_param;
    float* event_pos;
    float* event_dir;
    unsigned long long* counters;
    unsigned long long* ticket;
    const uint32_t* order;  // ticket -> photon index (TRAINING), or null
    int width;              // lanes of a wave that take photons; below 64, once
};

// Order buckets: more expected events first.
constexpr int kOrderBuckets = 128;
constexpr int kOrderChunk = 4096;  // photons per block of the sort kernels

// Parameters of training photon id (the walk kernel draws the same block).
__device__ __forceinline__ void training_params(const WalkArgs& a, uint64_t id, float& st, float& g, float& phi) {
    const uint4 pw = make_rng(a.seed, MS_TAG_WALK_PARAM, id).block(0);
    const bool focus = u24(pw.w) <= a.focus_thr;
    st = (focus ? a.fst_lo : a.st_lo) * __builtin_amdgcn_exp2f(u01(pw.x) * (focus ? a.fst_log2_ratio : a.st_log2_ratio));
    g = __builtin_fmaf(focus ? a.fg_span : a.g_span, u01(pw.y), focus ? a.fg_lo : a.g_lo);
    phi = __builtin_fmaf(a.a_span, u01(pw.z), a.a_lo);
}

// Bucket of the expected chain length, about 1 + tau + tau^2 (1 - g) / 3
// events for optical radius tau (a diffusion estimate; only its order matters),
// reversed so that bucket 0 holds the longest chains.
__device__ __forceinline__ int order_bucket(float st, float g) {
    const float cost = 1.0f + st + 0.35f * st * st * (1.0f - g);
    const int b = (int)(8.0f * __builtin_amdgcn_logf(cost));
    return kOrderBuckets - 1 - (b < 0 ? 0 : b > kOrderBuckets - 1 ? kOrderBuckets - 1 : b);
}

__global__ __launch_bounds__(256) void walk_order_count(const WalkArgs a, uint32_t* counts) {
    __shared__ uint32_t h[kOrderBuckets];
    for (int b = threadIdx.x; b < kOrderBuckets; b += blockDim.x) h[b] = 0u;
    __syncthreads();
    const uint64_t lo = (uint64_t)blockIdx.x * kOrderChunk;
    for (uint64_t i = lo + threadIdx.x; i < a.n && i < lo + kOrderChunk; i += blockDim.x) {
        float st, g, phi;
        training_params(a, a.photon_offset + i, st, g, phi);
        atomicAdd(&h[order_bucket(st, g)], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kOrderBuckets; b += blockDim.x)
        if (h[b]) atomicAdd(&counts[b], h[b]);
}

__global__ __launch_bounds__(256) void walk_order_scatter(const WalkArgs a, const uint32_t* counts, uint32_t* cursor,
                                                          uint32_t* order) {
    __shared__ uint32_t h[kOrderBuckets], base[kOrderBuckets], first[kOrderBuckets];
    __shared__ uint8_t key[kOrderChunk];
    for (int b = threadIdx.x; b < kOrderBuckets; b += blockDim.x) h[b] = 0u;
    if (threadIdx.x < 64) {
        // where each bucket starts: every block adds the counts up for itself
        const uint32_t c0 = counts[2 * threadIdx.x], c1 = counts[2 * threadIdx.x + 1];
        uint32_t incl = c0 + c1;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t v = __shfl_up(incl, off);
            if ((int)threadIdx.x >= off) incl += v;
        }
        first[2 * threadIdx.x] = incl - c0 - c1;
        first[2 * threadIdx.x + 1] = incl - c1;
    }
    __syncthreads();
    const uint64_t lo = (uint64_t)blockIdx.x * kOrderChunk;
    for (uint64_t i = lo + threadIdx.x; i < a.n && i < lo + kOrderChunk; i += blockDim.x) {
        float st, g, phi;
        training_params(a, a.photon_offset + i, st, g, phi);
        const int b = order_bucket(st, g);
        key[i - lo] = (uint8_t)b;
        atomicAdd(&h[b], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kOrderBuckets; b += blockDim.x) {
        base[b] = h[b] ? first[b] + atomicAdd(&cursor[b], h[b]) : 0u;
        h[b] = 0u;
    }
    __syncthreads();
    for (uint64_t i = lo + threadIdx.x; i < a.n && i < lo + kOrderChunk; i += blockDim.x) {
        const int b = key[i - lo];
        order[base[b] + atomicAdd(&h[b], 1u)] = (uint32_t)i;
    }
}

__device__ __forceinline__ void put3(float* base, uint64_t n, uint64_t i, V3 v) {
    if (!base) return;
    base[i] = v.x;
    base[n + i] = v.y;
    base[2 * n + i] = v.z;
}

// A photon's end (writing its record) and the start of the next one run in
// one pass per wave once this many lanes wait, or when no lane is walking, so
// that the code is not issued every iteration for a few lanes.
constexpr int kWalkRestartMin = 16;

// Chains a wave has left, with no photons to take, when it starts to walk
// them together.
constexpr int kWalkTogether = 16;

// What the events of the chains walked together draw: G consecutive events
// for each of 64 / G chains, four padding entries after each chain's.
struct alignas(16) WalkLds {
    float4 turn[128];   // mu, sin theta, cosine and sine of the azimuth
    float flight[128];  // flight length (inf: absorbed)
    float pick[128];    // uniform of the event choice
    float safe[32];     // per four events: |x|^2 below which none of them can leave the sphere
    uint32_t lane[64];  // lane that holds the k-th live chain
};

template <int MODE>
__global__ __launch_bounds__(256) void walk_kernel(const WalkArgs a) {
    __shared__ WalkLds lds_all[4];
    __shared__ BlockTotals totals;
    totals.reset();
    TicketPool pool;
    pool.reset((uint64_t)blockIdx.x * 4 + uniform_u32(threadIdx.x >> 6), (uint64_t)gridDim.x * 4, a.width, a.n);
    // lane state: walking, ended (record not yet written), idle, done
    bool active = false, ended = false, done = lane_id() >= a.width;
    bool absorbed = false, truncated = false;
    uint64_t i = 0;
    Rng rng = make_rng(a.seed, MS_TAG_WALK_EVENT, 0);
    V3 x = v3(0, 0, 0), d = v3(0, 0, 1), xk = v3(0, 0, 0), wk = v3(0, 0, 1);
    uint32_t nev = 0, c0 = 0, k = 1;
    float st = a.sigma_t, inv_st = 1.0f / a.sigma_t, g = a.g, phi = a.albedo, inv_phi = 1.0f, resv = 0.0f;
    Hg hg = hg_const(a.g);
    const float r = MODE == MS_WALK_ANALOG ? a.radius : 1.0f;
    const float r2 = MODE == MS_WALK_ANALOG ? a.r2 : 1.0f;
    uint64_t n_events = 0, n_abs = 0, n_trunc = 0, n_max = 0;

    // The record of a finished photon; x, d: where it ended and its direction.
    auto finish = [&](uint32_t nev, bool absorbed, bool truncated, V3 x, V3 d) __attribute__((always_inline)) {
        n_events += nev;
        n_abs += absorbed;
        n_trunc += truncated;
        n_max = nev > n_max ? nev : n_max;
        const uint64_t n = a.n;
        if (a.params) {
            put3(a.params, n, i, v3(MODE == MS_WALK_ANALOG ? a.st_report : st, g, phi));
        }
        if (a.n_scatter) a.n_scatter[i] = nev;
        if (a.absorbed) a.absorbed[i] = (uint8_t)absorbed;
        if (a.truncated) a.truncated[i] = (uint8_t)truncated;
        put3(a.exit_pos, n, i, x);
        put3(a.exit_dir, n, i, d);
        // exit frame of Sec. 4.1 after rotating by -psi about w_in = z
        const float ir = 1.0f / r;
        const V3 xh = ir * x;
        const float sin_t = __builtin_sqrtf(__builtin_fmaf(xh.x, xh.x, xh.y * xh.y));
        float cp = 1.0f, sp = 0.0f;
        if (sin_t > 0.0f) {
            cp = xh.x / sin_t;
            sp = xh.y / sin_t;
        }
        // fused products written out: this code is inlined twice
        auto turned = [&](V3 v) __attribute__((always_inline)) {
            return v3(__builtin_fmaf(v.y, sp, v.x * cp), __builtin_fmaf(v.y, cp, -(v.x * sp)), v.z);
        };
        if (a.exit_param) {
            const V3 wp = turned(d);
            put3(a.exit_param, n, i, v3(xh.z, wp.y, __builtin_fmaf(wp.x, xh.z, -(wp.z * sin_t))));
        }
        if (MODE == MS_WALK_TRAINING) {
            if (a.event_index) a.event_index[i] = k;
            put3(a.event_pos, n, i, turned(ir * xk));
            put3(a.event_dir, n, i, turned(wk));
        }
    };

    // The last chains of a wave, walked together.  A launch ends with a few
    // long chains (2 x 10^5 events of one photon in 2^22), each an event after
    // the other on a lane of its own: bound by the instructions of one event,
    // whatever lanes are idle.  Two thirds of those do not depend on where the
    // photon is: here a chain has G = 64 / (chains left) lanes, each draws
    // one of its next G events, and then all of them walk the G events on the
    // same state, reading the draws from LDS.  One wave issues an instruction
    // every 6 cycles: an event took 0.43 us alone and takes 0.11 (about 38
    // instructions, nearly all of them the turn of the direction); 2^22
    // training walks 105 -> 54 to 68 ms by seed and run, 2^16 73 -> 25 ms.
    auto walk_together = [&]() __attribute__((always_inline)) {
        WalkLds& L = lds_all[threadIdx.x >> 6];
        const int lane = lane_id();
        bool leader = true;  // of the lanes that hold one chain, the one that writes its record
        for (uint64_t live = ballot(active); live != 0; live = ballot(active && leader)) {
            const int n_live = __popcll(live);
            const int lg = n_live > 1 ? 6 - (32 - __builtin_clz((uint32_t)(n_live - 1))) : 6;
            const int G = 1 << lg, chain = lane >> lg, slot0 = chain * (G + 4);
            if (active && leader) L.lane[rank_in(live)] = (uint32_t)lane;
            wave_sync();
            const int src = (int)L.lane[chain < n_live ? chain : 0];
            wave_sync();
            auto from = [src](uint32_t v) __attribute__((always_inline)) { return (uint32_t)__shfl((int)v, src); };
            auto fromf = [src](float v) __attribute__((always_inline)) { return __shfl(v, src); };
            i = (uint64_t)from((uint32_t)i) | (uint64_t)from((uint32_t)(i >> 32)) << 32;
            rng.s0 = from(rng.s0);
            rng.s1 = from(rng.s1);
            rng.s2 = from(rng.s2);
            c0 = from(c0);
            nev = from(nev);
            k = from(k);
            x = v3(fromf(x.x), fromf(x.y), fromf(x.z));
            d = v3(fromf(d.x), fromf(d.y), fromf(d.z));
            xk = v3(fromf(xk.x), fromf(xk.y), fromf(xk.z));
            wk = v3(fromf(wk.x), fromf(wk.y), fromf(wk.z));
            st = fromf(st);
            inv_st = fromf(inv_st);
            g = fromf(g);
            if (MODE == MS_WALK_TRAINING) hg = hg_const(g);
            phi = fromf(phi);
            inv_phi = fromf(inv_phi);
            resv = fromf(resv);
            active = chain < n_live;
            leader = (lane & (G - 1)) == 0;
            // the draw that stands for "kept" under uniform weighting is 0
            // (else inf), against a reservoir that stays 1
            const bool uniform = a.weighting == MS_EVENT_UNIFORM;
            const float grow = uniform ? 0.0f : inv_phi;
            if (uniform) resv = 0.0f;
            // steps until the first chain reaches max_events, at most G at once
            uint32_t left = active ? a.max_events - nev : 0xFFFFFFFFu;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                const uint32_t o = (uint32_t)__shfl_xor((int)left, off);
                left = o < left ? o : left;
            }
            left = uniform_u32(left);
            int n_now = n_live;
            do {
                const uint32_t steps = left < (uint32_t)G ? left : (uint32_t)G;
                const uint32_t mine = (uint32_t)(lane & (G - 1));
                const uint4 w = rng.block(c0 + mine);
                const HgSample h = hg_sample(hg, u01(w.y));
                const float az = u01(w.z);
                float l = -flight_ln(u01(w.x)) * inv_st, u = 0.0f;
                if (MODE == MS_WALK_ANALOG) {
                    // the flight of a survivor is finite, so that infinity
                    // means absorbed alone (a medium can be as good as empty:
                    // its photons leave, however far they would have flown)
                    l = active && u24(w.w) > a.surv_thr ? INFINITY : __builtin_fminf(l, 0x1.fffffep127f);
                } else if (uniform) {
                    u = (uint64_t)u24(w.w) * (nev + mine + 1u) <= (1ull << 24) ? 0.0f : INFINITY;
                } else {
                    u = u01(w.w);
                }
                L.turn[slot0 + mine] = make_float4(h.mu, h.sin_t, cos_rev(az), sin_rev(az));
                L.flight[slot0 + mine] = l;
                L.pick[slot0 + mine] = u;
                // the flights of four events end to end, rounded up
                float l4 = l + __shfl_xor(l, 1);
                l4 += __shfl_xor(l4, 2);
                const float room = 0.9999f * r - l4;
                if ((lane & 3) == 0) L.safe[lane >> 2] = !active ? INFINITY : room > 0.0f ? room * room : 0.0f;
                wave_sync();
                // The reservoir only grows (to a rounding): none of these
                // events is chosen if none would be against its present value,
                // and past 2^24 no uniform of any later one is small enough.
                const bool choose = MODE == MS_WALK_TRAINING && ballot(active && u * resv <= 1.0001f) != 0;
                const bool grown = MODE == MS_WALK_ANALOG || ballot(active && !(resv > 0x1p25f)) == 0;
                // where a chain that leaves in these steps ends
                bool left_now = false, gone = false;
                uint32_t n_end = 0;
                V3 xe = x, de = d;
                auto step = [&](uint32_t e) __attribute__((always_inline)) {
                    const float4 t = L.turn[slot0 + e];
                    const float l = L.flight[slot0 + e];
                    if (MODE == MS_WALK_TRAINING) {
                        resv = __builtin_fmaf(resv, grow, 1.0f);
                        if (active && L.pick[slot0 + e] * resv <= 1.0f) {
                            xk = x;
                            wk = d;
                            k = nev + e + 1u;
                        }
                    }
                    const V3 dn = turn(d, t.x, t.y, t.z, t.w);
                    const V3 xn = fma3(l, dn, x);
                    if (active && !(dot(xn, xn) < r2)) {
                        active = false;
                        left_now = true;
                        n_end = nev + e + 1u;
                        gone = MODE == MS_WALK_ANALOG && l == INFINITY;
                        xe = gone ? x : fma3(sphere_exit(x, dn, r2), dn, x);
                        de = gone ? d : dn;
                    }
                    x = xn;
                    d = dn;
                };
                // Four events at a time without looking; where one of them is
                // chosen, or may leave the sphere and does, one by one.
                uint32_t e = 0;
                const float4* tp = L.turn + slot0;
                const float4* lp = reinterpret_cast<const float4*>(L.flight + slot0);
                const float* sp = L.safe + (chain << lg >> 2);
                for (; e + 4u <= steps; e += 4u) {
                    const float4 t0 = tp[0], t1 = tp[1], t2 = tp[2], t3 = tp[3], lq = *lp;
                    const float safe = *sp;
                    tp += 4;
                    ++lp;
                    ++sp;
                    const V3 d0 = turn(d, t0.x, t0.y, t0.z, t0.w), x0 = fma3(lq.x, d0, x);
                    const V3 d1 = turn(d0, t1.x, t1.y, t1.z, t1.w), x1 = fma3(lq.y, d1, x0);
                    const V3 d2 = turn(d1, t2.x, t2.y, t2.z, t2.w), x2 = fma3(lq.z, d2, x1);
                    const V3 d3 = turn(d2, t3.x, t3.y, t3.z, t3.w), x3 = fma3(lq.w, d3, x2);
                    bool look = ballot(!(dot(x, x) < safe)) != 0;
                    if (look)
                        look = ballot(active && !(dot(x0, x0) < r2 && dot(x1, x1) < r2 && dot(x2, x2) < r2 && dot(x3, x3) < r2)) != 0;
                    if (look || choose) {
#pragma unroll 1
                        for (uint32_t q = 0; q < 4; ++q) step(e + q);
                    } else {
                        x = x3;
                        d = d3;
                        if (!grown) {
#pragma unroll
                            for (int q = 0; q < 4; ++q) resv = __builtin_fmaf(resv, grow, 1.0f);
                        }
                    }
                }
#pragma unroll 1
                for (; e < steps; ++e) step(e);
                nev += steps;
                c0 += steps;
                left -= steps;
                bool cut = false;
                if (left == 0 && active && nev >= a.max_events) {
                    active = false;
                    left_now = cut = true;
                    n_end = nev;
                    xe = x;
                    de = d;
                }
                if (left_now && leader) finish(n_end, gone, cut, xe, de);
                n_now = __popcll(ballot(active && leader));
                wave_sync();
            } while (left != 0 && (2 * n_now > 64 / G || (G == 64 && n_now > 0)));
        }
    };

    bool due = true;
    for (;;) {
        if (due) {
            if (ended) {
                // x holds the exit point
                ended = false;
                finish(nev, absorbed, truncated, x, d);
            }
            const bool need = !active && !done;
            const uint64_t t = pool.take(need, a.ticket, a.width, a.n);
            if (need) {
                if (t < a.n) {
                    i = a.order ? a.order[t] : t;
                    active = true;
                    const uint64_t id = a.photon_offset + i;
                    rng = make_rng(a.seed, MS_TAG_WALK_EVENT, id);
                    if (MODE == MS_WALK_TRAINING) {
                        training_params(a, id, st, g, phi);
                        inv_st = 1.0f / st;
                        hg = hg_const(g);
                        // finite, so that the reservoir's first step gives 1
                        inv_phi = __builtin_fminf(1.0f / phi, 0x1.fffffep127f);
                    }
                    x = v3(0, 0, 0);
                    d = v3(0, 0, 1);
                    xk = x;
                    wk = d;
                    nev = 0;
                    c0 = 0;
                    k = 1;
                    resv = 0.0f;
                } else {
                    done = true;
                }
            }
            if (ballot(!done) == 0) break;
            if (pool.dry && __popcll(ballot(!done)) <= kWalkTogether) {
                walk_together();
                break;
            }
        }
        if (active) {
            ++nev;
            const uint4 w = rng.block(c0++);
            bool stop = false;
            absorbed = false;
            truncated = false;
            V3 xe = x;
            if (MODE == MS_WALK_ANALOG) {
                if (u24(w.w) > a.surv_thr) {
                    absorbed = true;
                    stop = true;
                }
            } else {
                bool keep;
                if (a.weighting == MS_EVENT_UNIFORM) {
                    keep = (uint64_t)u24(w.w) * nev <= (1ull << 24);
                } else {
                    resv = __builtin_fmaf(resv, inv_phi, 1.0f);
                    keep = u01(w.w) * resv <= 1.0f;
                }
                if (keep) {
                    xk = x;
                    wk = d;
                    k = nev;
                }
            }
            if (!stop) {
                const HgSample h = hg_sample(hg, u01(w.y));
                d = scatter(d, h.mu, h.sin_t, u01(w.z));
                const float l = -flight_ln(u01(w.x)) * inv_st;
                const V3 xn = fma3(l, d, x);
                if (!(dot(xn, xn) < r2)) {
                    xe = fma3(sphere_exit(x, d, r2), d, x);
                    stop = true;
                } else {
                    x = xn;
                    if (nev >= a.max_events) {
                        truncated = true;
                        xe = x;
                        stop = true;
                    }
                }
            }
            if (stop) {
                active = false;
                ended = true;
                x = xe;
            }
        }
        const uint64_t rmask = ballot(!active && !done);
        due = rmask != 0 && (__popcll(rmask) >= kWalkRestartMin || ballot(active) == 0);
    }
    if (a.counters) {
        const uint64_t v[4] = {wave_sum_u64(n_events), wave_sum_u64(n_abs), wave_sum_u64(n_trunc), wave_max_u64(n_max)};
        totals.add<true>(v, a.counters);
    }
}

// The ticket counter past the tickets that the waves begin with, and zeros
// after it.
__global__ void walk_ticket_kernel(unsigned long long* p, int n, uint64_t first) {
    const int t = threadIdx.x;
    if (t < n) p[t] = t == 0 ? first : 0ull;
}

}  // namespace msst

extern "C" {

ms_status ms_random_walk_workspace_size(const ms_walk_desc* desc, size_t* bytes) {
    MS_REQUIRE(desc != nullptr && bytes != nullptr, "ms_random_walk_workspace_size: NULL argument");
    // ticket counter; for training walks of fewer than 2^32 photons also the
    // order buckets, their cursors and the photon order (4 bytes per photon)
    *bytes = 256;
    if (desc->mode == MS_WALK_TRAINING && desc->n_photons < (1ull << 32))
        *bytes = 2048 + msst::align_up((size_t)desc->n_photons * 4, 256);
    return MS_OK;
}

ms_status ms_random_walk(const ms_walk_desc* desc, const ms_walk_out* out, void* workspace_dev,
                         size_t workspace_bytes, void* stream) {
    using namespace msst;
    MS_REQUIRE(desc != nullptr && out != nullptr, "ms_random_walk: NULL descriptor");
    const ms_walk_desc& d = *desc;
    MS_REQUIRE(d.n_photons > 0 && d.n_photons < (1ull << 40), "ms_random_walk: n_photons must be in [1, 2^40)");
    MS_REQUIRE(d.mode == MS_WALK_ANALOG || d.mode == MS_WALK_TRAINING, "ms_random_walk: unknown mode %d", d.mode);
    MS_REQUIRE(d.blocks_per_cu >= 0 && d.blocks_per_cu <= 64, "ms_random_walk: blocks_per_cu must be in [0, 64]");
    if (d.mode == MS_WALK_ANALOG) {
        MS_REQUIRE(d.sigma_t > 0.0 && d.sigma_t < 1e30, "ms_random_walk: sigma_t must be positive and finite");
        MS_REQUIRE(d.g > -1.0 && d.g < 1.0, "ms_random_walk: |g| must be < 1");
        MS_REQUIRE(d.albedo >= 0.0 && d.albedo <= 1.0, "ms_random_walk: albedo must be in [0, 1]");
        MS_REQUIRE(d.radius > 0.0 && d.radius < 1e30, "ms_random_walk: radius must be positive and finite");
    } else {
        MS_REQUIRE(d.event_weighting == MS_EVENT_ALBEDO_POWER || d.event_weighting == MS_EVENT_UNIFORM,
                   "ms_random_walk: unknown event weighting %d", d.event_weighting);
        MS_REQUIRE(d.st_range[0] > 0.0 && d.st_range[1] >= d.st_range[0] && d.st_range[1] < 1e30,
                   "ms_random_walk: st_range must satisfy 0 < lo <= hi");
        MS_REQUIRE(d.g_range[0] > -1.0 && d.g_range[1] >= d.g_range[0] && d.g_range[1] < 1.0,
                   "ms_random_walk: g_range must satisfy -1 < lo <= hi < 1");
        MS_REQUIRE(d.albedo_range[0] > 0.0 && d.albedo_range[1] >= d.albedo_range[0] && d.albedo_range[1] <= 1.0,
                   "ms_random_walk: albedo_range must satisfy 0 < lo <= hi <= 1");
        MS_REQUIRE(d.focus_fraction >= 0.0 && d.focus_fraction <= 1.0, "ms_random_walk: focus_fraction must be in [0, 1]");
        if (d.focus_fraction > 0.0) {
            MS_REQUIRE(d.focus_st_range[0] > 0.0 && d.focus_st_range[1] >= d.focus_st_range[0] &&
                           d.focus_st_range[1] < 1e30,
                       "ms_random_walk: focus_st_range must satisfy 0 < lo <= hi");
            MS_REQUIRE(d.focus_g_range[0] > -1.0 && d.focus_g_range[1] >= d.focus_g_range[0] && d.focus_g_range[1] < 1.0,
                       "ms_random_walk: focus_g_range must satisfy -1 < lo <= hi < 1");
        }
    }
    size_t ws_need = 0;
    ms_random_walk_workspace_size(desc, &ws_need);
    MS_REQUIRE(workspace_dev != nullptr, "ms_random_walk: workspace is NULL");
    if (workspace_bytes < ws_need)
        return set_error(MS_ERR_WORKSPACE_TOO_SMALL, "ms_random_walk: workspace needs %zu bytes", ws_need);
    MS_REQUIRE(((uintptr_t)workspace_dev & 7u) == 0, "ms_random_walk: workspace must be 8-byte aligned");

    int cus = 0;
    ms_status st = device_cu_count(&cus);
    if (st != MS_OK) return st;

    WalkArgs a{};
    a.seed = d.seed;
    a.photon_offset = d.photon_offset;
    a.n = d.n_photons;
    a.sigma_t = (float)d.sigma_t;
    a.g = (float)d.g;
    a.albedo = (float)d.albedo;
    a.radius = (float)d.radius;
    a.r2 = (float)d.radius * (float)d.radius;
    a.st_report = (float)(d.sigma_t * d.radius);
    a.surv_thr = (uint32_t)floor(d.albedo * 16777216.0);
    a.st_lo = (float)d.st_range[0];
    a.st_log2_ratio = (float)log2(d.st_range[1] / d.st_range[0]);
    a.g_lo = (float)d.g_range[0];
    a.g_span = (float)(d.g_range[1] - d.g_range[0]);
    a.a_lo = (float)d.albedo_range[0];
    a.a_span = (float)(d.albedo_range[1] - d.albedo_range[0]);
    a.focus_thr = (uint32_t)floor(d.focus_fraction * 16777216.0);
    if (d.focus_fraction > 0.0) {
        a.fst_lo = (float)d.focus_st_range[0];
        a.fst_log2_ratio = (float)log2(d.focus_st_range[1] / d.focus_st_range[0]);
        a.fg_lo = (float)d.focus_g_range[0];
        a.fg_span = (float)(d.focus_g_range[1] - d.focus_g_range[0]);
    }
    a.weighting = d.event_weighting;
    a.max_events = d.max_events ? d.max_events : (1u << 20);
    a.params = out->params;
    a.n_scatter = out->n_scatter;
    a.event_index = out->event_index;
    a.absorbed = out->absorbed;
    a.truncated = out->truncated;
    a.exit_pos = out->exit_pos;
    a.exit_dir = out->exit_dir;
    a.exit_param = out->exit_param;
    a.event_pos = out->event_pos;
    a.event_dir = out->event_dir;
    a.counters = reinterpret_cast<unsigned long long*>(out->counters);
    a.ticket = reinterpret_cast<unsigned long long*>(workspace_dev);

    // Three blocks (as many as fit) keep VALU issue busy: 2^24 training walks
    // in 119 / 101 / 114 ms with two / three / four.  At 2^22 the end of the
    // launch is half of it, and 54 to 71 ms are measured with one to eight, as
    // much by run and seed as by the number of blocks.
    const int bpc = d.blocks_per_cu ? d.blocks_per_cu : 3;
    // A few photons with long chains are spread over all waves: the fewer
    // chains a wave has, the sooner they walk together (2^16 training walks
    // 30 -> 25 ms, 4096 22 -> 9 ms).  Where even the longest chains are short
    // (the expected events of the thickest, most backward medium, as in
    // order_bucket, or the event and absorption limits) full waves finish
    // them sooner: 10^5 analog walks of 17 events 0.14 ms, spread 0.25 ms.
    const bool training = d.mode == MS_WALK_TRAINING;
    const bool focus = training && d.focus_fraction > 0.0;
    const double tau = training ? fmax(d.st_range[1], focus ? d.focus_st_range[1] : 0.0) : d.sigma_t * d.radius;
    const double g_lo = training ? fmin(d.g_range[0], focus ? d.focus_g_range[0] : 1.0) : d.g;
    double longest = fmin(1.0 + tau + 0.35 * tau * tau * (1.0 - g_lo), (double)a.max_events);
    if (!training && d.albedo < 1.0) longest = fmin(longest, 1.0 / (1.0 - d.albedo));
    a.width = 8;
    while (a.width < 64 && d.n_photons > (uint64_t)a.width * 4 * cus * bpc) a.width *= 2;
    if (longest < 256.0) a.width = d.n_photons <= (uint64_t)16 * 4 * cus ? 16 : 64;
    uint64_t blocks = (d.n_photons + 4 * a.width - 1) / (4 * a.width);
    if (blocks > (uint64_t)cus * bpc) blocks = (uint64_t)cus * bpc;
    const uint64_t first = blocks * 4 * a.width;
    hipStream_t s = (hipStream_t)stream;
    if (ws_need > 256) {
        // longest expected chains first: counts, prefix, scatter of the ids
        uint32_t* counts = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(workspace_dev) + 1024);
        uint32_t* cursor = counts + kOrderBuckets;
        uint32_t* order = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(workspace_dev) + 2048);
        const unsigned ob = (unsigned)((d.n_photons + kOrderChunk - 1) / kOrderChunk);
        hipLaunchKernelGGL(walk_ticket_kernel, dim3(1), dim3(256), 0, s, a.ticket, 128 + kOrderBuckets, first);
        hipLaunchKernelGGL(walk_order_count, dim3(ob), dim3(256), 0, s, a, counts);
        hipLaunchKernelGGL(walk_order_scatter, dim3(ob), dim3(256), 0, s, a, (const uint32_t*)counts, cursor, order);
        a.order = order;
    } else {
        hipLaunchKernelGGL(walk_ticket_kernel, dim3(1), dim3(64), 0, s, a.ticket, 1, first);
    }
    MS_LAUNCHED();
    if (d.mode == MS_WALK_ANALOG)
        hipLaunchKernelGGL(walk_kernel<MS_WALK_ANALOG>, dim3((unsigned)blocks), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(walk_kernel<MS_WALK_TRAINING>, dim3((unsigned)blocks), dim3(256), 0, s, a);
    MS_LAUNCHED();
    clear_error();
    return MS_OK;
}

}  // extern "C"
