// device.hpp -- gfx950 device primitives of libmsst: counter-based RNG,
// scattering sampling, frames, wave-level helpers and bfloat16 / FP8 packing.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace msst {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds, each two
// 32x32 -> 64-bit products; the key advances by the Weyl increments between
// rounds.  Counter = (draw index, id low, id high, stream tag).
//
// A lane draws many blocks of one id.  The draw index enters the first round
// on one side only, so the other side's product, and one product of the
// second round, depend on the id alone: a stream holds what the third round
// needs of them (s0, s1, s2) in place of the id, and a block takes 18 of the
// 20 products.  A round's two exclusive ors are one v_bitop3_b32 each.  The
// walk and the render loops are bound by VALU issue, and a 32 x 32 -> 64-bit
// product issues like a fused multiply-add (4.7 to 5 cycles of 2.4 GHz a wave
// measured, transcendentals 9.7), so instructions are what counts: with the
// shorter uniform and logarithm below, 2^22 training walks 117 -> 105 ms, the
// 512^2 x 256 spp sphere and box image 15.4 -> 14.9 ms (plain, sigma_t 40) and
// 16.0 -> 15.0 ms (learned, sigma_t 80).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return (uint32_t)__builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
constexpr uint32_t kPhiloxM0 = 0xD2511F53u, kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u, kPhiloxW1 = 0xBB67AE85u;

struct Rng {
    uint32_t k0, k1, tag;
    uint32_t s0, s1, s2;
    // Words of block c0.
    __device__ __forceinline__ uint4 block(uint32_t c0) const {
        const uint64_t p0 = (uint64_t)kPhiloxM0 * c0;
        const uint64_t p1 = (uint64_t)kPhiloxM1 * ((uint32_t)(p0 >> 32) ^ (tag ^ k1));
        uint32_t x0 = (uint32_t)(p1 >> 32) ^ s0, x1 = (uint32_t)p1, x2 = (uint32_t)p0 ^ s1, x3 = s2;
#pragma unroll
        for (int round = 2; round < 10; ++round) {
            const uint64_t q0 = (uint64_t)kPhiloxM0 * x0, q1 = (uint64_t)kPhiloxM1 * x2;
            x0 = xor3((uint32_t)(q1 >> 32), x1, k0 + round * kPhiloxW0);
            x1 = (uint32_t)q1;
            x2 = xor3((uint32_t)(q0 >> 32), x3, k1 + round * kPhiloxW1);
            x3 = (uint32_t)q0;
        }
        return make_uint4(x0, x1, x2, x3);
    }
};

__device__ __forceinline__ Rng make_rng(uint64_t seed, uint32_t tag, uint64_t id) {
    Rng r;
    r.k0 = (uint32_t)seed;
    r.k1 = (uint32_t)(seed >> 32);
    r.tag = tag;
    const uint64_t p1 = (uint64_t)kPhiloxM1 * (uint32_t)(id >> 32);
    const uint64_t p0 = (uint64_t)kPhiloxM0 * ((uint32_t)(p1 >> 32) ^ (uint32_t)id ^ r.k0);
    r.s0 = (uint32_t)p1 ^ (r.k0 + kPhiloxW0);
    r.s1 = (uint32_t)(p0 >> 32) ^ (r.k1 + kPhiloxW1);
    r.s2 = (uint32_t)p0;
    return r;
}

// Uniform on (0, 1]: ((w >> 8) + 1) 2^-24, exact in binary32.
__device__ __forceinline__ float u01(uint32_t w) { return __builtin_fmaf((float)(w >> 8), 0x1p-24f, 0x1p-24f); }
// 24-bit integer form k = (w >> 8) + 1 of the same uniform, for exact
// integer decisions (u <= p  <=>  k <= floor(p 2^24)).
__device__ __forceinline__ uint32_t u24(uint32_t w) { return (w >> 8) + 1u; }

// Hardware transcendentals: v_log_f32 / v_exp_f32 work in base 2,
// v_sin_f32 / v_cos_f32 take revolutions.
__device__ __forceinline__ float fast_ln(float x) { return __builtin_amdgcn_logf(x) * 0.69314718055994531f; }
__device__ __forceinline__ float fast_exp(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504088896341f); }
__device__ __forceinline__ float sin_rev(float r) { return __builtin_amdgcn_sinf(r); }
__device__ __forceinline__ float cos_rev(float r) { return __builtin_amdgcn_cosf(r); }
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float fast_rsq(float x) { return __builtin_amdgcn_rsqf(x); }
// Hardware square root and quotient through the reciprocal (1 ulp each)
// where a correctly rounded result buys nothing: the IEEE sequences cost
// about ten instructions apiece.
__device__ __forceinline__ float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ float fast_div(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }

// Natural log for free-flight lengths -log(u) / sigma_t, about 1 ulp: the
// hardware log2 times ln 2 in two parts, the product's rounding taken up by
// fused steps.  Constants and order are those into which LLVM's AMDGPU back end
// expands logf, so that the value is logf's for every uniform u in [2^-24, 1]
// (compared for all of them), without its scaling of denormals and its test
// for infinities.
__device__ __forceinline__ float flight_ln(float u) {
    const float y = __builtin_amdgcn_logf(u), hi = 0x1.62e42ep-1f, lo = 0x1.efa39ep-25f;
    const float r = y * hi;
    return __builtin_fmaf(y, hi, __builtin_fmaf(y, lo, __builtin_fmaf(y, hi, -r)));
}

// Box-Muller pair from two uniforms.
__device__ __forceinline__ void box_muller(float ua, float ub, float& n0, float& n1) {
    const float r = fast_sqrt(-2.0f * fast_ln(ua));
    n0 = r * cos_rev(ub);
    n1 = r * sin_rev(ub);
}

// Henyey-Greenstein sample for uniform xi (Eq. 1 importance sampling),
// returned as (mu, sin theta).  The inverse CDF mu(xi) is evaluated through
//   1 - mu = 2 (1 - g)^2 (1 - xi)(1 + g xi) / q^2,
//   1 + mu = 2 (1 + g)^2 xi (1 - g + g xi) / q^2,    q = 1 + g (2 xi - 1),
// which carry no cancellation for any g (including 0) or xi, so that both
// mu and sin(theta) = sqrt((1 - mu)(1 + mu)) keep full relative precision
// in the strongly forward and backward tails.
struct HgSample {
    float mu, sin_t;
};
// What a medium's asymmetry g alone decides of the phase function: one medium
// per launch or photon, so its loops hold these and no more arithmetic on g.
struct Hg {
    float g, omg, om2, op2;     // g, 1 - g, 2 (1 - g)^2, 2 (1 + g)^2
    float eval_c, eval_a, eval_b;  // (1 - g^2) / 4 pi, -2 g, 1 + g^2
};
__host__ __device__ __forceinline__ Hg hg_const(float g) {
    Hg h;
    h.g = g;
    h.omg = 1.0f - g;
    const float opg = 1.0f + g;
    h.om2 = 2.0f * h.omg * h.omg;
    h.op2 = 2.0f * opg * opg;
    h.eval_c = 0.0795774715459476679f * __builtin_fmaf(-g, g, 1.0f);
    h.eval_a = -2.0f * g;
    h.eval_b = __builtin_fmaf(g, g, 1.0f);
    return h;
}
__device__ __forceinline__ HgSample hg_sample(const Hg& c, float xi) {
    const float q = __builtin_fmaf(c.g, __builtin_fmaf(xi, 2.0f, -1.0f), 1.0f);
    const float iq2 = fast_rcp(q * q);
    const float om = c.om2 * (1.0f - xi) * __builtin_fmaf(c.g, xi, 1.0f) * iq2;
    const float opq = c.op2 * xi * __builtin_fmaf(c.g, xi, c.omg);
    const float op = opq * iq2;
    HgSample h;
    h.mu = __builtin_fminf(1.0f, __builtin_fmaxf(-1.0f, 0.5f * __builtin_fmaf(opq, iq2, -om)));
    h.sin_t = fast_sqrt(__builtin_fminf(1.0f, om * op));
    return h;
}

// HG phase function value (Eq. 1).
__device__ __forceinline__ float hg_eval(const Hg& c, float cos_t) {
    const float den = __builtin_fmaf(c.eval_a, cos_t, c.eval_b);
    return c.eval_c * fast_rsq(den) * fast_rcp(den);
}

struct V3 {
    float x, y, z;
};
__device__ __forceinline__ V3 v3(float x, float y, float z) { return V3{x, y, z}; }
__device__ __forceinline__ V3 operator+(V3 a, V3 b) { return v3(a.x + b.x, a.y + b.y, a.z + b.z); }
__device__ __forceinline__ V3 operator-(V3 a, V3 b) { return v3(a.x - b.x, a.y - b.y, a.z - b.z); }
__device__ __forceinline__ V3 operator*(float s, V3 a) { return v3(s * a.x, s * a.y, s * a.z); }
// Fused in one order, so that every loop that evaluates it rounds alike.
__device__ __forceinline__ float dot(V3 a, V3 b) {
    return __builtin_fmaf(a.z, b.z, __builtin_fmaf(a.x, b.x, a.y * b.y));
}
__device__ __forceinline__ V3 fma3(float s, V3 a, V3 b) {
    return v3(__builtin_fmaf(s, a.x, b.x), __builtin_fmaf(s, a.y, b.y), __builtin_fmaf(s, a.z, b.z));
}
__device__ __forceinline__ V3 normalize(V3 a) { return fast_rsq(dot(a, a)) * a; }
__device__ __forceinline__ V3 cross(V3 a, V3 b) {
    return v3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}

// Right-handed orthonormal basis (b1, b2, n) of Duff et al., "Building an
// Orthonormal Basis, Revisited", JCGT 2017.
__device__ __forceinline__ void onb(V3 n, V3& b1, V3& b2) {
    const float sign = __builtin_copysignf(1.0f, n.z);
    const float a = -fast_rcp(sign + n.z);
    const float b = n.x * n.y * a;
    b1 = v3(1.0f + sign * n.x * n.x * a, sign * b, -sign * n.x);
    b2 = v3(b, sign + n.y * n.y * a, -n.y);
}

// Direction with polar cosine mu (sine s) and azimuth cosine ca, sine sa about
// d: the rotation in the frame of onb(), with the order and the fused products
// written out (and no others fused, also where one turn follows another), so
// that every loop that turns a direction rounds alike.  The sign that onb()
// takes from d.z is moved through the products, where it is exact, to sa and to
// the result's z.
__device__ __forceinline__ float times_sign(float v, float of) {
    return __uint_as_float(__float_as_uint(v) ^ (__float_as_uint(of) & 0x80000000u));
}
__device__ __forceinline__ V3 turn(V3 d, float mu, float s, float ca, float sa) {
#pragma clang fp contract(off)
    const float az = __builtin_fabsf(d.z);
    const float a = fast_rcp(1.0f + az);
    const float b = (d.x * d.y) * -a;
    const float b1x = __builtin_fmaf(-a, d.x * d.x, 1.0f), b2y = __builtin_fmaf(-(d.y * d.y), a, 1.0f);
    const float ss = times_sign(sa, d.z);
    const float tx = __builtin_fmaf(b, ss, b1x * ca), ty = __builtin_fmaf(b, ca, b2y * ss);
    const float tz = __builtin_fmaf(-d.x, ca, -(d.y * ss));
    const float nx = __builtin_fmaf(tx, s, d.x * mu), ny = __builtin_fmaf(ty, s, d.y * mu), nz = __builtin_fmaf(tz, s, az * mu);
    const float il = fast_rsq(__builtin_fmaf(nz, nz, __builtin_fmaf(nx, nx, ny * ny)));
    return v3(nx * il, ny * il, times_sign(nz * il, d.z));
}

// Direction with polar cosine mu (sine s) and azimuth (revolutions) about d.
__device__ __forceinline__ V3 scatter(V3 d, float mu, float s, float az_rev) {
    return turn(d, mu, s, cos_rev(az_rev), sin_rev(az_rev));
}

// Distance from x (inside) along unit d to the sphere |y|^2 = r2 about the
// origin: the positive root of t^2 + 2 b t - delta = 0, delta = r2 - |x|^2,
// taken in the form without cancellation.
__device__ __forceinline__ float sphere_exit(V3 x, V3 d, float r2) {
    const float b = dot(x, d);
    const float delta = __builtin_fmaxf(0.0f, r2 - dot(x, x));
    const float root = fast_sqrt(__builtin_fmaf(b, b, delta));
    return b >= 0.0f ? fast_div(delta, b + root) : root - b;
}

// Softplus log(1 + e^x) = max(x, 0) + log(1 + e^-|x|) and its derivative.
// The larger of x and 0 is a median with infinity, one instruction; a maximum
// first quiets x, and the compiler turns a median back into one unless it does
// not see the infinity.
__device__ __forceinline__ float softplus(float x) {
    float inf = __builtin_inff();
    asm("" : "+s"(inf));
    return __builtin_amdgcn_fmed3f(x, 0.0f, inf) + fast_ln(1.0f + fast_exp(-__builtin_fabsf(x)));
}
__device__ __forceinline__ float sigmoid(float x) { return fast_rcp(1.0f + fast_exp(-x)); }

// ---------------------------------------------------------------------------
// Wave helpers (64 lanes).
__device__ __forceinline__ int lane_id() { return __lane_id(); }
__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }
__device__ __forceinline__ int rank_in(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}
__device__ __forceinline__ uint32_t uniform_u32(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t uniform_u64(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Per-wave ticket pool over a global 64-bit counter: lanes that need work
// take consecutive tickets from the wave's private range and the wave
// refills it with one atomic per `chunk` tickets.  Wave w begins with tickets
// w chunk .. w chunk + chunk - 1 and the counter past those of all waves; a
// wave that has seen the end of the tickets asks no more: on one counter,
// thousands of waves would wait for each other's atomics at either end.
struct TicketPool {
    uint64_t next, end;
    bool dry;
    __device__ __forceinline__ void reset(uint64_t wave, uint64_t waves, uint32_t chunk, uint64_t n) {
        next = wave * chunk;
        end = next + chunk;
        dry = waves * chunk >= n;
    }
    // Returns this lane's ticket (meaningful where `need`): work for it below n.
    __device__ __forceinline__ uint64_t take(bool need, unsigned long long* counter, uint32_t chunk, uint64_t n) {
        const uint64_t mask = ballot(need);
        if (mask == 0) return 0;
        const uint32_t n_need = (uint32_t)__popcll(mask);
        const uint32_t rank = (uint32_t)rank_in(mask);
        const uint64_t avail = end - next;
        uint64_t mine;
        if (avail >= n_need) {
            mine = next + rank;
            next += n_need;
        } else {
            unsigned long long base = n;
            if (!dry) {
                const int leader = __ffsll((long long)mask) - 1;
                if (lane_id() == leader) base = atomicAdd(counter, (unsigned long long)chunk);
                base = uniform_u64(__shfl(base, leader));
                dry = base + chunk >= n;
            }
            mine = rank < avail ? next + rank : base + (rank - avail);
            next = base + (n_need - avail);
            end = base + chunk;
        }
        return mine;
    }
};

// Wave-wide sum of a 64-bit counter (result valid in every lane).
__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        uint64_t o = __shfl_xor(v, off);
        v = o > v ? o : v;
    }
    return v;
}

// A launch's totals: the waves of a block add theirs up in LDS, and the last
// one to finish adds the block's to the global counters.  One atomic per wave
// and counter, all on one cache line, took 60 us of a launch of 1500 waves.
struct BlockTotals {
    unsigned long long sum[4];
    uint32_t finished;
    // Every thread of the block, before the first add.
    __device__ __forceinline__ void reset() {
        if (threadIdx.x < 4) sum[threadIdx.x] = 0ull;
        if (threadIdx.x == 0) finished = 0u;
        __syncthreads();
    }
    // Once per wave, with its totals (the same in every lane): v[0..2] are
    // added to the counters, v[3] is added or, with kMax, their maximum taken.
    template <bool kMax>
    __device__ __forceinline__ void add(const uint64_t* v, unsigned long long* counters) {
        if (lane_id() != 0) return;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (kMax && q == 3) atomicMax(&sum[q], (unsigned long long)v[q]);
            else if (v[q]) atomicAdd(&sum[q], (unsigned long long)v[q]);
        }
        __threadfence_block();
        if (atomicAdd(&finished, 1u) != blockDim.x / 64 - 1) return;
        __threadfence_block();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned long long t = sum[q];
            if (t == 0) continue;
            if (kMax && q == 3) atomicMax(counters + q, t);
            else atomicAdd(counters + q, t);
        }
    }
};

// ---------------------------------------------------------------------------
// bfloat16 (round to nearest even) and FP8 E4M3 (OCP) conversions.
__device__ __forceinline__ uint16_t bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

}  // namespace msst
