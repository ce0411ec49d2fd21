// Nucleus (top-p) transform of logit rows: device code (included by mpv.hip).
//
// Sec. 4.1 names the setting (nucleus sampling with top-p 0.9 and 0.99); the definition taken
// is the usual one.  With p = softmax(z / T): keep the smallest set {v : z_v >= tau}, tau one
// of the row's values, whose mass reaches top_p; every other token gets the logit -inf, so that
// whatever reads the row afterwards sees the renormalised truncated distribution.  Tokens with
// equal logits are kept or dropped together.
//
// One workgroup per row.  Masses are 2^((z - m) log2(e)/T), m the row's maximum: the largest is 1.
//   1. One sweep over the row adds up its mass and copies the tokens that can matter, those
//      whose probability is within 2^-12 of the largest, into a list in LDS (value and position).
//   2. If they reach top_p and fit, the row is never looked at again: it is filled with -inf while
//      tau is found among the listed tokens by bisection over the order-preserving integer keys of
//      float values (each probe returns the mass of {z >= cut} and the nearest values on either
//      side of the cut, to which the bracket snaps), and the kept tokens are put back: the row is read
//      once and written once.
//      (If the list did not fit only because the largest logit comes late, it is made again, in a second sweep.)
//   3. Otherwise (flat rows, top_p close to 1) the mass of the row is sorted into bins of 1/32
//      binary order by logit (a second sweep); the bin that contains tau is known then, and a third
//      sweep writes the row, keeping what lies above the bin, dropping what lies below, and
//      listing the bin's own tokens, among which tau is found as in 2.
//   4. Where a bin holds more tokens than the list (thousands of equal or nearly equal logits), its tokens are sorted into
//      bins again, by key, until one key is left, and the row is written in a sweep of its own.
// What bounds it: traffic, at the rate of a device copy.  10 496 rows of 151 936 bf16 logits, top_p 0.9 held by
// a few dozen tokens: 1.25 ms = 5.1 TB/s read and written (a large copy reaches 5.1); it was 2.11 ms with a read for
// the maximum, one for the list and one for the masked copy.  960 rows of 128 256: 115 us, was 350.  Flat rows
// (top_p 0.99, 40 000 tokens kept; 3): 191 us, was 925 with every probe a pass over the row.  Rows of 32 000 to 50 000
// times the same logit are the ones that took less with those probes (960 of 32 000 in bf16: 62 us, now 68).
// The list is filled best if the first cut is good: from the maximum of the workgroup's first 4 vectors per lane
// (32 768 bf16 logits), which are in registers anyway; from one vector per lane the same rows took 143 us.
//
// Whether the list suffices depends on when the waves hear of each other's maxima (a list that fills up
// before the largest logit is known is given up), the results do not (bitwise reproducible): all of these
// ways compare the same two numbers.  top_p of the row's mass comes from the first sweep, whose sums are
// added in a fixed order against references that do not depend on timing.  The mass of an upper set is a sum of
// whole units (2^-40), exact in any order where the list could have been used: 4096 terms or less of 24 bits
// within 2^-12 of the largest.  (In the bins a token counts with its mass rounded down to a whole unit: an upper set
// appears smaller by V * 2^-40 of the largest mass at most.)

#pragma once

#include "mpv_device.h"

namespace mpv {

constexpr int kNucleusUnroll = 4;     // 16-byte loads in flight per lane
// Rows of this many vectors or more get a workgroup of 1024 lanes (two per compute unit), shorter ones 256
// (eight).  Measured, 1024 / 256 lanes: 960 rows of 16 032 vectors 115 / 177 us, 300 of 8 000 40 / 53, 30 of
// 16 032 22 / 93; 960 of 4 000 69 / 56, 2 000 of 125 54 / 18, 64 of 128 12 / 9: the line is drawn where few
// rows still gain (a row's own time counts) and many do not lose much.
constexpr int kNucleusLongRow = 2048;

// ascending unsigned key of a float (no NaN): negative values reversed, sign bit flipped
__device__ __forceinline__ uint32_t float_key(float f) {
    const uint32_t b = __float_as_uint(f + 0.0f);            // -0 -> +0
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key_float(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}


// Barrier between waves that hand each other values through LDS only: row loads and stores in
// flight are not waited for.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Keys of row values, as dense as the type's values (bf16: the upper half of the float's key says it all).
template <class E> struct RowKey;
template <> struct RowKey<ElemF32> {
    __device__ static __forceinline__ uint32_t of(float z) { return float_key(z); }
    __device__ static __forceinline__ float value(uint32_t k) { return key_float(k); }
};
template <> struct RowKey<ElemBF16> {
    __device__ static __forceinline__ uint32_t of(float z) { return float_key(z) >> 16; }
    __device__ static __forceinline__ float value(uint32_t k) { return key_float((k << 16) | ((k & 0x8000u) ? 0u : 0xffffu)); }
};

// What one probe of the bisection finds out about a cut.
struct NucleusProbe {
    double mass;            // of {z >= cut}
    float below, above;     // largest z < cut, smallest z >= cut
    int count;              // |{z >= cut}|
};

// The list has room for this many tokens per wave, 2 KB each: 33 KB for 16 waves.  (With twice the room only
// one workgroup of 1024 lanes ran per compute unit: 143 against 118 us on the rows above.)
constexpr int kNucleusPerWave = 256;
constexpr float kNucleusSpan = 12.f;                   // listed: within this many binary orders of the largest
constexpr double kNucleusUnit = 1099511627776.0;       // 2^40
constexpr int kNucleusBins = 1280;                     // of 1/32 binary order; the last one takes the rest
constexpr float kBinsPerOctave = 32.f;

template <int BLOCK>
struct NucleusShared {
    static constexpr int NW = BLOCK / kWave;
    static constexpr int CAP = NW * kNucleusPerWave;
    // Several copies of the bins, a lane adds to one of them: on rows of few distinct logits a wave's additions to one bin
    // are performed one after the other.  960 rows of 128 256 bf16 logits that are multiples of 2 (normal, standard deviation
    // 3): 549 us with one copy, 222 with four; rows without such logits take 1 % longer or less.  (With 256 lanes a
    // second copy would leave room for seven workgroups in a compute unit, not eight.)
    static constexpr int COPIES = BLOCK == 1024 ? 4 : 1;
    static constexpr int STRIDE = kNucleusBins + 2;    // (copies start in different LDS banks)
    union {
        struct { float z[CAP]; int at[CAP]; } list;
        alignas(16) unsigned long long bin[COPIES * STRIDE];      // the first copy has the sums in the end
    };
    double mass[NW];
    float lo[NW], hi[NW];
    int count[NW];
    int listed;                                        // by a sweep that lists what it knows to matter: tokens listed
    uint32_t max_key;                                  // key of the largest logit seen so far
    int tau_bin;
    double above_bin, want;                            // mass above that bin; top_p of the row's
    float tau;
    int kept;
};

// mass of a token in units of 2^-40, relative to the largest
__device__ __forceinline__ double nucleus_units(float z, float k32, float nA) {
    return floor(static_cast<double>(fast_exp2(fmaf(z, k32, nA))) * kNucleusUnit);
}

// A probe over the listed tokens by `LANES` lanes (a wave, or the whole workgroup).
template <int LANES>
__device__ __forceinline__ NucleusProbe probe_listed(const float* z, int n, float cut, float k32, float nA) {
    NucleusProbe p;
    p.mass = 0.0; p.below = -INFINITY; p.above = INFINITY; p.count = 0;
    for (int i = static_cast<int>(threadIdx.x) % LANES; i < n; i += LANES) {
        const float v = z[i];
        const bool in = v >= cut;
        p.mass += in ? nucleus_units(v, k32, nA) : 0.0;
        p.below = in ? p.below : fmaxf(p.below, v);
        p.above = in ? fminf(p.above, v) : p.above;
        p.count += in ? 1 : 0;
    }
    return p;
}
__device__ __forceinline__ int wave_sum_i32(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x124, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, true);
    return (__builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16)) +
           (__builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48));
}
__device__ __forceinline__ NucleusProbe wave_total(NucleusProbe p) {
    p.mass = wave_sum(p.mass);
    p.below = wave_max(p.below);
    p.above = -wave_max(-p.above);
    p.count = wave_sum_i32(p.count);
    return p;
}
template <int BLOCK>
__device__ __forceinline__ NucleusProbe block_total(NucleusProbe p, NucleusShared<BLOCK>& sh) {
    constexpr int NW = BLOCK / kWave;
    p = wave_total(p);
    const int w = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    lds_barrier();                                     // the previous results have been read
    if (lane == 0) { sh.mass[w] = p.mass; sh.lo[w] = p.below; sh.hi[w] = p.above; sh.count[w] = p.count; }
    lds_barrier();
    p.mass = sh.mass[0]; p.below = sh.lo[0]; p.above = sh.hi[0]; p.count = sh.count[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) {
        p.mass += sh.mass[i];
        p.below = fmaxf(p.below, sh.lo[i]);
        p.above = fminf(p.above, sh.hi[i]);
        p.count += sh.count[i];
    }
    return p;
}

// Bisection: the smallest upper set of row values whose mass reaches `want`, between the set of
// lo_key (which does, given by tau and kept) and hi_key (from which on nothing is left).  `base`: the
// mass of the tokens above those that the probes look at.
template <class PROBE>
__device__ __forceinline__ void nucleus_bisect(uint32_t lo_key, uint32_t hi_key, double base, double want, float& tau, int& kept, PROBE probe) {
    for (int step = 0; step < 40 && hi_key - lo_key > 1u; ++step) {
        const NucleusProbe p = probe(key_float(lo_key + (hi_key - lo_key) / 2u));
        if (base + p.mass >= want) {
            tau = p.above;                             // the same upper set, named by its smallest value
            kept = p.count;
            lo_key = float_key(tau);
        } else {
            hi_key = float_key(p.below) + 1u;          // every cut above `below` has this upper set or less
        }
    }
}
// ... among the listed tokens.  Up to 16 per lane the first wave does it alone: a probe is then
// a few hundred cycles without a barrier, and the other waves' stores of the row go on meanwhile.
// Four waves share more than 8 per lane while the compute units have idle slots (flat float32 rows of 1000: 8 rows
// 22.7 us by the first wave alone, 15.0 shared, 1024 rows 29.5 and 26.2; but 2000 with a few raised tokens 35.1 and 40.7).
template <int BLOCK>
__device__ __forceinline__ void bisect_listed(NucleusShared<BLOCK>& sh, int n, uint32_t lo_key, uint32_t hi_key, double base, double want,
                                              float k32, float nA, float& tau, int& kept) {
    const int alone = BLOCK == 256 && gridDim.x <= 1024u ? 8 : 16;
    if (n <= alone * kWave) {
        if (threadIdx.x < kWave) {
            nucleus_bisect(lo_key, hi_key, base, want, tau, kept, [&](float cut) __attribute__((always_inline)) {
                return wave_total(probe_listed<kWave>(sh.list.z, n, cut, k32, nA));
            });
            if (threadIdx.x == 0) { sh.tau = tau; sh.kept = kept; }
        }
        lds_barrier();
        tau = sh.tau;
        kept = sh.kept;
    } else {
        nucleus_bisect(lo_key, hi_key, base, want, tau, kept, [&](float cut) __attribute__((always_inline)) {
            return block_total<BLOCK>(probe_listed<BLOCK>(sh.list.z, n, cut, k32, nA), sh);
        });
    }
}

// A row of `V` elements: `head` elements before the first 16-byte boundary, nvec vectors, the rest.
template <class E>
struct NucleusRow {
    const typename E::T* z;
    typename E::T* o;
    int V, head, nvec, tail0;
    __device__ __forceinline__ NucleusRow(const typename E::T* z_, typename E::T* o_, int V_) : z(z_), o(o_), V(V_) {
        const int mis = static_cast<int>((reinterpret_cast<uintptr_t>(z) & 15u) / sizeof(typename E::T));
        head = mis ? min(E::VEC - mis, V) : 0;
        nvec = (V - head) / E::VEC;
        tail0 = head + nvec * E::VEC;
    }
    // Calls f(values, position of the first, raw vector, inside) for every vector, all lanes of a wave
    // together (lanes past the end: inside = false, -inf values), then edge(value, position, inside) for
    // the elements before and after.  U loads per lane are in flight: with 32 waves per compute unit (two
    // workgroups of 1024 lanes or eight of 256, 64 registers per lane) the other waves' work covers their latency.  begin(vectors) sees the
    // first U vectors of every lane before any of them is used.
    struct Nothing { template <class R> __device__ __forceinline__ void operator()(const R&) const {} };
    template <int BLOCK, int U, class F, class G, class H = Nothing>
    __device__ __forceinline__ void sweep(F f, G edge, H begin = H()) const {
        const int tid = threadIdx.x;
        const typename E::T* const base = z + head;
        for (int i0 = 0; i0 < nvec; i0 += BLOCK * U) {
            uint4 raw[U];
#pragma unroll
            for (int u = 0; u < U; ++u) raw[u] = load_raw_at(base, min(i0 + u * BLOCK + tid, nvec - 1));
            if (i0 == 0) begin(raw);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * BLOCK + tid;
                const bool inside = i < nvec;
                if (!inside) raw[u] = NegInfVec<E>::v();
                float a[E::VEC];
                E::unpack(raw[u], a);
                f(a, head + i * E::VEC, raw[u], inside);
            }
        }
        if (head > 0) {
            const bool inside = tid < head;
            edge(inside ? E::load_one_global(z + tid) : -INFINITY, tid, inside);
        }
        if (tail0 < V) {
            const bool inside = tail0 + tid < V;
            edge(inside ? E::load_one_global(z + tail0 + tid) : -INFINITY, tail0 + tid, inside);
        }
    }
    __device__ __forceinline__ void store_vec(int e, const uint4& v) const {
        typedef unsigned v4u __attribute__((ext_vector_type(4)));
        const v4u t = {v.x, v.y, v.z, v.w};
        *as_global(reinterpret_cast<v4u*>(o + e)) = t;
    }
};

template <class E> struct MaskedStore;
template <> struct MaskedStore<ElemF32> {
    __device__ static __forceinline__ float one(float z, float tau) { return z >= tau ? z : -INFINITY; }
    __device__ static __forceinline__ uint4 vec(const uint4& r, float tau) {
        uint4 o;
        o.x = __float_as_uint(one(__uint_as_float(r.x), tau)); o.y = __float_as_uint(one(__uint_as_float(r.y), tau));
        o.z = __float_as_uint(one(__uint_as_float(r.z), tau)); o.w = __float_as_uint(one(__uint_as_float(r.w), tau));
        return o;
    }
    __device__ static __forceinline__ float to_elem(float v) { return v; }
    __device__ static __forceinline__ uint4 pack(const float (&v)[4]) {
        return make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3]));
    }
};
template <> struct MaskedStore<ElemBF16> {
    static constexpr uint32_t kNegInf = 0xff80u;
    __device__ static __forceinline__ uint32_t word(uint32_t w, float tau) {
        const uint32_t lo = (__uint_as_float(w << 16) >= tau) ? (w & 0xffffu) : kNegInf;
        const uint32_t hi = (__uint_as_float(w & 0xffff0000u) >= tau) ? (w & 0xffff0000u) : (kNegInf << 16);
        return hi | lo;
    }
    __device__ static __forceinline__ uint4 vec(const uint4& r, float tau) {
        uint4 o;
        o.x = word(r.x, tau); o.y = word(r.y, tau); o.z = word(r.z, tau); o.w = word(r.w, tau);
        return o;
    }
    __device__ static __forceinline__ uint16_t to_elem(float v) { return static_cast<uint16_t>(__float_as_uint(v) >> 16); }
    __device__ static __forceinline__ uint32_t two(float lo, float hi) {       // (values that are bf16 numbers already)
        return (__float_as_uint(lo) >> 16) | (__float_as_uint(hi) & 0xffff0000u);
    }
    __device__ static __forceinline__ uint4 pack(const float (&v)[8]) {
        return make_uint4(two(v[0], v[1]), two(v[2], v[3]), two(v[4], v[5]), two(v[6], v[7]));
    }
};


// Per-wave part of the first sweep: the mass of what the wave has seen, against a reference that is
// the largest logit it has seen (or the largest of the workgroup's first vectors), and the wave's
// own run of the list (no atomic, no wait: a listed token costs a few instructions).
template <class E, int BLOCK>
struct NucleusCollect {
    NucleusShared<BLOCK>& sh;
    float k32, span;        // span: of what is listed, in units of the logits
    int first;              // the wave's run of the list starts here
    float mz, mk;           // the reference: mk = mz * k32, kFloor at least (the same in every lane of the wave)
    float top;              // the largest logit of any wave, as far as this one knows
    float cut, thr;         // listed: logits >= cut; a vector whose terms add up to less than thr has none
    float s;                // this lane's mass, in units of the reference
    int n;                  // tokens listed by this wave (more than fit: too many)
    __device__ __forceinline__ void init(float k, float top, int wave) {
        k32 = k; span = kNucleusSpan / k; first = wave * kNucleusPerWave;
        mz = top; mk = fmaxf(top * k, OnlineLse::kFloor);
        s = 0.f; n = 0;
        set_cut(top);
    }
    // what to list depends on the largest logit any wave has seen (asked for now and then: an old one
    // only means that more is listed than need be; what is within the span is sorted out at the end)
    __device__ __forceinline__ void refresh() {
        set_cut(uniform_f32(key_float(__hip_atomic_load(&sh.max_key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))));
    }
    __device__ __forceinline__ void set_cut(float largest) {
        top = largest;
        const bool none = !(top * k32 > OnlineLse::kFloor) || n > kNucleusPerWave;     // nothing but masked logits so far, or no room left
        cut = none ? INFINITY : top - span;
        // (0.98: the rounding of the terms; 0.9: a logit above the reference must always be noticed)
        thr = none ? 0.9f : fminf(0.9f, 0.98f * fast_exp2(fmaf(cut, k32, -mk)));
    }
    template <int COUNT>
    __device__ __forceinline__ float terms(const float (&a)[COUNT]) const {
        float t0 = fast_exp2(fmaf(a[0], k32, -mk)), t1 = COUNT > 1 ? fast_exp2(fmaf(a[COUNT > 1 ? 1 : 0], k32, -mk)) : 0.f;
#pragma unroll
        for (int i = 2; i + 1 < COUNT; i += 2) {
            t0 += fast_exp2(fmaf(a[i], k32, -mk));
            t1 += fast_exp2(fmaf(a[i + 1], k32, -mk));
        }
        return t0 + t1;
    }
    template <int COUNT>
    __device__ __forceinline__ void add(const float (&a)[COUNT], int e0) {
        float v = terms(a);
        if (__builtin_amdgcn_ballot_w64(!(v < thr)) != 0ull) {
            float lm = a[0];
#pragma unroll
            for (int i = 1; i < COUNT; ++i) lm = fmaxf(lm, a[i]);
            if (__builtin_amdgcn_ballot_w64(lm > mz) != 0ull) {        // a new largest logit
                const float nz = wave_max(lm), nmk = fmaxf(nz * k32, OnlineLse::kFloor);
                s *= fast_exp2(mk - nmk);
                mz = nz; mk = nmk;
                v = terms(a);
                if ((threadIdx.x & (kWave - 1)) == 0) atomicMax(&sh.max_key, float_key(nz));
                set_cut(fmaxf(nz, top));
            }
            if (cut < INFINITY) {
#pragma unroll
                for (int i = 0; i < COUNT; ++i) {
                    const unsigned long long hit = __builtin_amdgcn_ballot_w64(a[i] >= cut);
                    if (hit) {
                        const int mine = n + static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(hit >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(hit), 0u)));
                        if (a[i] >= cut && mine < kNucleusPerWave) { sh.list.z[first + mine] = a[i]; sh.list.at[first + mine] = e0 + i; }
                        n += __popcll(hit);
                    }
                }
            }
        }
        s += v;
    }
};

template <int BLOCK>
__device__ __forceinline__ void clear_bins(NucleusShared<BLOCK>& sh) {
    lds_barrier();                                     // what was in LDS has been read
    uint4* const pair = reinterpret_cast<uint4*>(sh.bin);
    for (int i = threadIdx.x; i < NucleusShared<BLOCK>::COPIES * NucleusShared<BLOCK>::STRIDE / 2; i += BLOCK) pair[i] = make_uint4(0u, 0u, 0u, 0u);
    lds_barrier();
}

// Adds the copies up and finds the bin that takes the mass `above` all bins to `want` (sh.tau_bin; sh.above_bin, the mass
// above it).  WHOLE: the bins hold the whole row, and `want` (out of reach by its rounding only if top_p is so close
// to 1 that no list reaches it either) is lowered to top_p of what they hold.  Otherwise they do reach it but for the rounding
// of other partial sums: the lowest that is not empty then.
template <int BLOCK, bool WHOLE>
__device__ __forceinline__ void find_bin(NucleusShared<BLOCK>& sh, double above, double& want, float top_p) {
    constexpr int COPIES = NucleusShared<BLOCK>::COPIES, STRIDE = NucleusShared<BLOCK>::STRIDE;
    const int lane = threadIdx.x & (kWave - 1);
    lds_barrier();
    if (COPIES > 1) {
        ulonglong2* const pair = reinterpret_cast<ulonglong2*>(sh.bin);
        for (int i = threadIdx.x; i < kNucleusBins / 2; i += BLOCK) {
            ulonglong2 t = pair[i];
#pragma unroll
            for (int c = 1; c < COPIES; ++c) { t.x += pair[c * STRIDE / 2 + i].x; t.y += pair[c * STRIDE / 2 + i].y; }
            pair[i] = t;
        }
        lds_barrier();
    }
    if (threadIdx.x < kWave) {
        constexpr int PER = kNucleusBins / kWave;
        static_assert(kNucleusBins % kWave == 0, "whole bins per lane");
        double mine = 0.0;
        for (int i = 0; i < PER; ++i) mine += static_cast<double>(sh.bin[lane * PER + i]);
        const double incl = wave_inclusive_scan(mine), up_to = __shfl_up(incl, 1, kWave);
        if (WHOLE) {
            const double whole = lane_f64(incl, kWave - 1);
            if (!(whole >= want)) want = static_cast<double>(top_p) * whole;
        }
        const unsigned long long some = __builtin_amdgcn_ballot_w64(mine > 0.0);
        const unsigned long long reach = some & __builtin_amdgcn_ballot_w64(above + incl >= want);
        if (lane == (reach ? __ffsll(static_cast<long long>(reach)) - 1 : some ? 63 - __clzll(static_cast<long long>(some)) : 0)) {
            double run = above + (lane > 0 ? up_to : 0.0);
            sh.tau_bin = lane * PER;                   // (there is a bin that is not empty, unless a logit is infinite)
            sh.above_bin = run;
            for (int i = 0; i < PER; ++i) {
                const double m = static_cast<double>(sh.bin[lane * PER + i]);
                if (m > 0.0) { sh.tau_bin = lane * PER + i; sh.above_bin = run; }
                run += m;
                if (run >= want) break;
            }
            sh.want = want;
        }
    }
    lds_barrier();
    want = sh.want;
}

// top_p in (0, 1): see the file header; keep_all: top_p = 1, nothing is dropped (tau = the row's
// minimum).  threshold_out / kept_out may be null.
template <class E, int BLOCK>
__global__ __launch_bounds__(BLOCK) void nucleus_kernel(const typename E::T* in, typename E::T* out, int V, float k32,
                                                        float top_p, int keep_all, float* threshold_out, int32_t* kept_out) {
    using T = typename E::T;
    __shared__ NucleusShared<BLOCK> sh;
    const int64_t r = blockIdx.x;
    const NucleusRow<E> row(in + r * V, out + r * V, V);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid & (kWave - 1);

    float tau = -INFINITY;                                    // so far: everything is kept
    int kept = V;
    bool written = false;
    float row_max = -INFINITY;
    double want = 0.0;                                        // top_p of the row's mass, in units
    if (!keep_all) {
        // ---- first sweep: the row's mass, its maximum, the list
        if (tid == 0) sh.max_key = float_key(-INFINITY);
        lds_barrier();
        NucleusCollect<E, BLOCK> c{sh};
        c.init(k32, -INFINITY, wave);
        int countdown = 0;
        row.template sweep<BLOCK, kNucleusUnroll>(
            [&](const float (&a)[E::VEC], int e0, const uint4&, bool) __attribute__((always_inline)) {
                if (countdown == 0) { c.refresh(); countdown = kNucleusUnroll; }
                --countdown;
                c.add(a, e0);
            },
            [&](float z, int e, bool) __attribute__((always_inline)) {
                const float a[1] = {z};
                c.add(a, e);
            },
            [&](const uint4 (&raw)[kNucleusUnroll]) __attribute__((always_inline)) {
                // every wave starts from the largest of the workgroup's first vectors
                float m = -INFINITY;
#pragma unroll
                for (int u = 0; u < kNucleusUnroll; ++u) {
                    float a[E::VEC];
                    E::unpack(raw[u], a);
#pragma unroll
                    for (int i = 0; i < E::VEC; ++i) m = fmaxf(m, a[i]);
                }
                m = wave_max(m);
                if (lane == 0) atomicMax(&sh.max_key, float_key(m));
                lds_barrier();
                c.init(k32, uniform_f32(key_float(sh.max_key)), wave);
                lds_barrier();                                // everybody starts from the same maximum
            });
        lds_barrier();                                        // the list and the maximum are complete
        row_max = uniform_f32(key_float(sh.max_key));
        const float nA = -row_max * k32;
        {   // the row's mass: each wave's part, brought to the row's maximum
            const double part = wave_sum(static_cast<double>(c.s)) * exp2(static_cast<double>(c.mk) + static_cast<double>(nA));
            NucleusProbe p;
            p.mass = lane == 0 ? part : 0.0; p.below = -INFINITY; p.above = INFINITY; p.count = 0;
            want = static_cast<double>(top_p) * block_total<BLOCK>(p, sh).mass * kNucleusUnit;
        }
        if (row_max * k32 > OnlineLse::kFloor) {              // (a row of masked logits only has nothing to drop)
            // what is within the span of the maximum moves to the front of the list
            const float cut0 = row_max - kNucleusSpan / k32;
            int listed = 0;
            bool complete = true;
            {
                constexpr int PER = kNucleusPerWave / kWave;
                float z[PER];
                int at[PER], within = 0;
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    const int j = i * kWave + lane;
                    z[i] = -INFINITY; at[i] = 0;
                    if (j < min(c.n, kNucleusPerWave)) { z[i] = sh.list.z[wave * kNucleusPerWave + j]; at[i] = sh.list.at[wave * kNucleusPerWave + j]; }
                    within += __popcll(__builtin_amdgcn_ballot_w64(z[i] >= cut0));
                }
                if (lane == 0) sh.count[wave] = c.n > kNucleusPerWave ? -1 : within;
                lds_barrier();                                // (and the runs have been read)
                int before = 0;
                for (int w = 0; w < NucleusShared<BLOCK>::NW; ++w) {
                    const int k = __builtin_amdgcn_readfirstlane(sh.count[w]);
                    if (k < 0) complete = false;
                    if (w < wave) before += k;
                    listed += k;
                }
                if (complete) {
#pragma unroll
                    for (int i = 0; i < PER; ++i) {
                        const unsigned long long in = __builtin_amdgcn_ballot_w64(z[i] >= cut0);
                        if (in) {
                            const int mine = before + static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(in >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(in), 0u)));
                            if (z[i] >= cut0) { sh.list.z[mine] = z[i]; sh.list.at[mine] = at[i]; }
                            before += __popcll(in);
                        }
                    }
                }
                lds_barrier();
            }
            NucleusProbe all;
            all.mass = -1.0;
            if (complete) all = block_total<BLOCK>(probe_listed<BLOCK>(sh.list.z, listed, cut0, k32, nA), sh);
            if (!complete && want <= 1.05 * kNucleusUnit) {
                // The runs were full before the largest token came, which has 95 % of what is needed or more: what is within
                // the span of it, listed in a sweep of its own.  (300 rows of 50 001 bf16 logits, normal with a standard
                // deviation of 2, one of 16 at four fifths of the row: by the bins 45 us, so 28.  A limit of 1.25 would
                // make rows 15 % slower whose list does not suffice after all.)
                if (tid == 0) sh.listed = 0;
                lds_barrier();
                auto list_one = [&](float z, int e) __attribute__((always_inline)) {
                    if (z >= cut0) {
                        const int at = atomicAdd(&sh.listed, 1);
                        if (at < NucleusShared<BLOCK>::CAP) { sh.list.z[at] = z; sh.list.at[at] = e; }
                    }
                };
                row.template sweep<BLOCK, 2>(
                    [&](const float (&a)[E::VEC], int e0, const uint4&, bool) __attribute__((always_inline)) {
#pragma unroll
                        for (int i = 0; i < E::VEC; ++i) list_one(a[i], e0 + i);
                    },
                    [&](float z, int e, bool) __attribute__((always_inline)) { list_one(z, e); });
                lds_barrier();
                listed = __builtin_amdgcn_readfirstlane(sh.listed);
                if (listed <= NucleusShared<BLOCK>::CAP) all = block_total<BLOCK>(probe_listed<BLOCK>(sh.list.z, listed, cut0, k32, nA), sh);
            }
            if (all.mass >= want) {
                // ---- tau is among the listed tokens: fill the row, find tau, put the kept tokens back
                const uint4 fill = NegInfVec<E>::v();
                for (int i = tid; i < row.nvec; i += BLOCK) row.store_vec(row.head + i * E::VEC, fill);
                if (tid < row.head) *as_global(row.o + tid) = MaskedStore<E>::to_elem(-INFINITY);
                if (row.tail0 + tid < V) *as_global(row.o + row.tail0 + tid) = MaskedStore<E>::to_elem(-INFINITY);
                tau = all.above;
                kept = all.count;
                bisect_listed<BLOCK>(sh, listed, float_key(tau), float_key(row_max) + 1u, 0.0, want, k32, nA, tau, kept);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this wave's share of the fill has been performed
                lds_barrier();                                        // ... and everybody's
                for (int i = tid; i < listed; i += BLOCK) {
                    const float z = sh.list.z[i];
                    if (z >= tau) *as_global(row.o + sh.list.at[i]) = MaskedStore<E>::to_elem(z);
                }
                written = true;
            } else {
                // ---- second sweep: the mass of every bin (bins are ordered as the logits are)
                clear_bins(sh);
                unsigned long long* const bin = sh.bin + (lane & (NucleusShared<BLOCK>::COPIES - 1)) * NucleusShared<BLOCK>::STRIDE;
                auto bin_of = [&](float y) __attribute__((always_inline)) -> int {
                    return static_cast<int>(fminf(fmaxf(-kBinsPerOctave * y, 0.f), kNucleusBins - 1.f));
                };
                auto units_of = [&](float y) __attribute__((always_inline)) -> unsigned long long {
                    return static_cast<unsigned long long>(fast_exp2(y) * static_cast<float>(kNucleusUnit));
                };
                if (want > (2.0 / 3.0) * static_cast<double>(top_p) * kNucleusUnit * static_cast<double>(V)) {
                    // On average a token has two thirds of the largest one's mass or more: the row is nearly level.
                    // Each lane adds in a register for as long as its tokens are of one bin.  960 rows of 128 256 equal
                    // bf16 logits: 239 us without, 205; on a row that is not level it costs 5 % (normal, standard
                    // deviation 1: 211 us without, 222).
                    int held_bin = 0;
                    unsigned long long held = 0ull;
                    auto into_bin = [&](float z) __attribute__((always_inline)) {
                        const float y = fmaf(z, k32, nA);
                        const int b = bin_of(y);
                        if (b != held_bin) {
                            if (held) atomicAdd(&bin[held_bin], held);
                            held_bin = b;
                            held = 0ull;
                        }
                        held += units_of(y);
                    };
                    row.template sweep<BLOCK, 2>(
                        [&](const float (&a)[E::VEC], int, const uint4&, bool) __attribute__((always_inline)) {
#pragma unroll
                            for (int i = 0; i < E::VEC; ++i) into_bin(a[i]);
                        },
                        [&](float z, int, bool) __attribute__((always_inline)) { into_bin(z); });
                    if (held) atomicAdd(&bin[held_bin], held);
                } else {
                    auto into_bin = [&](float z) __attribute__((always_inline)) {
                        const float y = fmaf(z, k32, nA);
                        const int b = bin_of(y);
                        const unsigned long long units = units_of(y);
                        if (units) atomicAdd(&bin[b], units);
                    };
                    row.template sweep<BLOCK, 2>(
                        [&](const float (&a)[E::VEC], int, const uint4&, bool) __attribute__((always_inline)) {
#pragma unroll
                            for (int i = 0; i < E::VEC; ++i) into_bin(a[i]);
                        },
                        [&](float z, int, bool) __attribute__((always_inline)) { into_bin(z); });
                }
                find_bin<BLOCK, true>(sh, 0.0, want, top_p);
                const int tb = __builtin_amdgcn_readfirstlane(sh.tau_bin);
                double above_bin = sh.above_bin;
                // how many tokens the bin holds at most: its mass over the smallest a token of it can have
                // (one unit less for each token's rounding down)
                bool fits = tb < kNucleusBins - 1;
                if (fits) {
                    const double least = floor(static_cast<double>(fast_exp2(-(static_cast<float>(tb) + 1.01f) / kBinsPerOctave)) * kNucleusUnit) - 1.0;
                    fits = least >= 1.0 && static_cast<double>(sh.bin[tb]) <= least * NucleusShared<BLOCK>::CAP;
                }
                lds_barrier();                                // the bins have been read
                if (fits) {
                    // ---- third sweep: write the row, list the bin's tokens (dropped for now)
                    if (tid == 0) sh.listed = 0;
                    lds_barrier();
                    const float lo_y = tb > 0 ? static_cast<float>(tb) : -INFINITY, hi_y = static_cast<float>(tb) + 1.f;
                    int above = 0;
                    auto place = [&](float z, int e, bool inside) __attribute__((always_inline)) -> bool {      // true: kept
                        const float y = -kBinsPerOctave * fmaf(z, k32, nA);
                        const bool in_bin = inside && y >= lo_y && y < hi_y;
                        if (in_bin) {
                            const int at = atomicAdd(&sh.listed, 1);
                            if (at < NucleusShared<BLOCK>::CAP) { sh.list.z[at] = z; sh.list.at[at] = e; }
                        }
                        const bool keep = inside && y < lo_y;
                        above += keep ? 1 : 0;
                        return keep;
                    };
                    row.template sweep<BLOCK, 2>(
                        [&](const float (&a)[E::VEC], int e0, const uint4& raw, bool inside) __attribute__((always_inline)) {
                            float m[E::VEC];
#pragma unroll
                            for (int i = 0; i < E::VEC; ++i) m[i] = place(a[i], e0 + i, inside) ? a[i] : -INFINITY;
                            if (inside) row.store_vec(e0, MaskedStore<E>::pack(m));
                            (void)raw;
                        },
                        [&](float z, int e, bool inside) __attribute__((always_inline)) {
                            const bool keep = place(z, e, inside);
                            if (inside) *as_global(row.o + e) = MaskedStore<E>::to_elem(keep ? z : -INFINITY);
                        });
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    NucleusProbe p;
                    p.mass = 0.0; p.below = -INFINITY; p.above = INFINITY; p.count = above;
                    const int count_above = block_total<BLOCK>(p, sh).count;      // (its barriers also complete the list)
                    const int n = min(__builtin_amdgcn_readfirstlane(sh.listed), NucleusShared<BLOCK>::CAP);
                    const NucleusProbe bin = block_total<BLOCK>(probe_listed<BLOCK>(sh.list.z, n, -INFINITY, k32, nA), sh);
                    tau = bin.above;
                    kept = bin.count;
                    bisect_listed<BLOCK>(sh, n, float_key(tau), float_key(row_max) + 1u, above_bin, want, k32, nA, tau, kept);
                    kept += count_above;
                    for (int i = tid; i < n; i += BLOCK) {
                        const float z = sh.list.z[i];
                        if (z >= tau) *as_global(row.o + sh.list.at[i]) = MaskedStore<E>::to_elem(z);
                    }
                    written = true;
                } else {
                    // ---- too many tokens in one bin: its ends, then bins again, by key, until one key is left.  960 rows of
                    // 128 256 logits with a standard deviation of 0.01: 326 us in bf16, 610 in float32; with a bisection
                    // whose probes read the row 1 190 and 1 880.
                    const float lo_y = tb > 0 ? static_cast<float>(tb) : -INFINITY, hi_y = tb < kNucleusBins - 1 ? static_cast<float>(tb) + 1.f : INFINITY;
                    NucleusProbe ends;
                    ends.mass = 0.0; ends.below = -INFINITY; ends.above = INFINITY; ends.count = 0;
                    auto end = [&](float z) __attribute__((always_inline)) {
                        const float y = -kBinsPerOctave * fmaf(z, k32, nA);
                        const bool in_bin = y >= lo_y && y < hi_y;            // (never a logit of -inf)
                        ends.below = in_bin ? fmaxf(ends.below, z) : ends.below;
                        ends.above = in_bin ? fminf(ends.above, z) : ends.above;
                    };
                    row.template sweep<BLOCK, 2>(
                        [&](const float (&a)[E::VEC], int, const uint4&, bool) __attribute__((always_inline)) {
#pragma unroll
                            for (int i = 0; i < E::VEC; ++i) end(a[i]);
                        },
                        [&](float z, int, bool) __attribute__((always_inline)) { end(z); });
                    ends = block_total<BLOCK>(ends, sh);
                    uint32_t lo_key = RowKey<E>::of(uniform_f32(ends.above)), hi_key = RowKey<E>::of(uniform_f32(ends.below));
                    while (lo_key < hi_key) {
                        int shift = 0;
                        while (((hi_key - lo_key) >> shift) >= static_cast<uint32_t>(kNucleusBins)) ++shift;
                        clear_bins(sh);
                        auto into_bin = [&](float z) __attribute__((always_inline)) {
                            const uint32_t key = RowKey<E>::of(z);
                            if (key >= lo_key && key <= hi_key) atomicAdd(&bin[(hi_key - key) >> shift], units_of(fmaf(z, k32, nA)));
                        };
                        row.template sweep<BLOCK, 2>(
                            [&](const float (&a)[E::VEC], int, const uint4&, bool) __attribute__((always_inline)) {
#pragma unroll
                                for (int i = 0; i < E::VEC; ++i) into_bin(a[i]);
                            },
                            [&](float z, int, bool) __attribute__((always_inline)) { into_bin(z); });
                        find_bin<BLOCK, false>(sh, above_bin, want, top_p);
                        above_bin = sh.above_bin;
                        hi_key -= static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(sh.tau_bin)) << shift;
                        lo_key = max(lo_key, hi_key - ((1u << shift) - 1u));
                    }
                    tau = RowKey<E>::value(lo_key);
                }
            }
        }
    }
    if (!written) {
        // ---- masked copy (in place if out == in: every element is read and written by the same lane)
        NucleusProbe p;
        p.mass = 0.0; p.below = -INFINITY; p.above = INFINITY; p.count = 0;
        row.template sweep<BLOCK, kNucleusUnroll>(
            [&](const float (&a)[E::VEC], int e0, const uint4& raw, bool inside) __attribute__((always_inline)) {
                if (inside) {
                    row.store_vec(e0, MaskedStore<E>::vec(raw, tau));
#pragma unroll
                    for (int i = 0; i < E::VEC; ++i) p.count += a[i] >= tau ? 1 : 0;
                }
            },
            [&](float z, int e, bool inside) __attribute__((always_inline)) {
                if (inside) {
                    *as_global(row.o + e) = MaskedStore<E>::to_elem(z >= tau ? z : -INFINITY);
                    p.count += z >= tau ? 1 : 0;
                }
            });
        kept = block_total<BLOCK>(p, sh).count;
    }
    if (tid == 0) {
        if (threshold_out) threshold_out[r] = tau;
        if (kept_out) kept_out[r] = kept;
    }
}

}  // namespace mpv
