// Walk of the top-vertex pipeline (top.h): for every vertex x, the wedges
// x - y - w with y and w below x are counted per endpoint w in LDS, and x
// adds C(a,2) + C(b,2) per endpoint.
//
// Most wedges belong to few hubs with thousands of middles (on the power-law
// graph of 20M edges 600 vertices hold 2.1e9 of 3.35e9), so a band of
// endpoint ranks is counted by a whole workgroup whose waves need no barrier
// between them: each wave takes chunks of 64 middles on its own (a lane per
// middle: the slice of its list inside the band), flattens the slices by a
// prefix sum over its lanes and adds to the shared counters by LDS atomics.
// Only the band's reduction and clearing are barriers.
//
// Flattening: 64 GP positions at a time, GP consecutive ones per lane.  Every
// non-empty slice marks its first position with lane + 1 (one LDS byte), a
// running maximum (GP - 1 per lane, one DPP scan) gives each position its
// slice, and one LDS word per slice (list start minus first position, with
// the sign of the anchor edge in bit 31) turns it into the list entry to load.
#include "band.h"
#include "top.h"

namespace bbc {

// LDS of one wave's flattening: one mark byte per position of a group (zero
// between groups), and per slice (list start - first position) mod 2^30 |
// sign << 31.
template <int GP>
struct FlatLds {
    uint32_t mark[GP / 4 * kWave];
    uint32_t tab[kWave];
};

// The slices of a wave's lanes, laid end to end.
struct Flat {
    int32_t total;      // positions
    int32_t ex, len;    // this lane's slice: first position, length
    uint32_t carry;     // slice (+ 1) holding the last position of the groups before
};

// One group of positions: entries and slice words (GP consecutive positions
// per lane; the sign of the anchor edge is bit 31 of the slice word) and how
// many of this lane's positions hold a wedge.  full (the same for every
// lane): all of them do.
template <int GP>
struct Group {
    uint32_t x[GP], tv[GP];
    uint32_t sl[GP];  // slices (lanes) of the positions
    int32_t nv;
    bool full;
};

// Loads the entries of a group whose slice words are known: position j + i of
// slice word tv lies at (tv + j + i) mod 2^30.  Every lane loads (the first
// entry of all where it has no wedge): the number of loads in flight is the
// same on every path, so a later wait for an older group need not wait for
// this one.
template <int GP>
__device__ __forceinline__ void load_entries(const uint32_t* __restrict__ ent, int32_t j, Group<GP>& g) {
    uint32_t off[GP];  // byte offsets: the shift drops the sign
#pragma unroll
    for (int i = 0; i < GP; ++i) off[i] = (g.tv[i] + (uint32_t)(j + i)) << 2;
    if (!g.full) {
#pragma unroll
        for (int i = 0; i < GP; ++i) off[i] = i < g.nv ? off[i] : 0u;
    }
#pragma unroll
    for (int i = 0; i < GP; ++i)
        g.x[i] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(ent) + off[i]);
}

// Lays the lanes' slices [st, st + len) of ent (sign: bit 31 of e) end to end.
__device__ __forceinline__ void flat_begin(Flat& f, uint32_t* __restrict__ tab, uint32_t st, int32_t len,
                                           uint32_t e) {
    const int32_t inc = (int32_t)wave_inclusive_sum_dpp((uint32_t)len);
    f.total = __builtin_amdgcn_readlane(inc, kWave - 1);
    f.len = len;
    f.ex = inc - len;
    f.carry = 0;
    __builtin_amdgcn_wave_barrier();
    tab[lane_id()] = ((st - (uint32_t)f.ex) & 0x3fffffffu) | (e & 0x80000000u);
    __builtin_amdgcn_wave_barrier();
}

// Loads the group at position j0 (groups in order).
template <int GP>
__device__ __forceinline__ void flat_load(Flat& f, uint32_t* __restrict__ mark, const uint32_t* __restrict__ tab,
                                          const uint32_t* __restrict__ ent, int32_t j0, Group<GP>& g) {
    const int lane = lane_id();
    const uint32_t d = (uint32_t)(f.ex - j0);
    if (f.len > 0 && d < (uint32_t)(GP * kWave)) reinterpret_cast<unsigned char*>(mark)[d] = (unsigned char)(lane + 1);
    __builtin_amdgcn_wave_barrier();
    static_assert(GP == 4, "a lane's marks are one word");
    const uint32_t w = mark[lane];
    mark[lane] = 0u;
    __builtin_amdgcn_wave_barrier();
    uint32_t k[GP];
#pragma unroll
    for (int i = 0; i < GP; ++i) k[i] = (w >> (8 * i)) & 255u;
#pragma unroll
    for (int i = 1; i < GP; ++i) k[i] = max(k[i], k[i - 1]);
    const uint32_t inc = wave_inclusive_max_dpp(k[GP - 1]);
    // exclusive: the lane before (wave_shr:1), lane 0 takes 0
    const uint32_t before =
        max((uint32_t)__builtin_amdgcn_update_dpp(0, (int)inc, 0x138, 0xf, 0xf, false), f.carry);
    f.carry = max(f.carry, (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1));
    const int32_t j = j0 + lane * GP;
    g.nv = f.total - j;
    g.full = j0 + GP * kWave <= f.total;
#pragma unroll
    for (int i = 0; i < GP; ++i) {
        g.sl[i] = (max(k[i], before) - 1u) & (kWave - 1);
        g.tv[i] = tab[g.sl[i]];
    }
    load_entries<GP>(ent, j, g);
}

// Where a band keeps the counter of endpoint rank r, wedge type t: slot =
// r * kSlotMul mod the band's slots (see band.h).  The multiplier is scaled so
// that the product's bits under wmask are the byte offset of the word; the
// bits below it (fm) pick the slot inside the word, the type moved from bit 31
// by ts to bit tm the field inside the slot.  Modes 0-2 differ in these numbers
// only, which sit in scalar registers; mode 3 (one word per slot and type) has
// the type in the byte offset.
struct BandFields {
    uint32_t mul, wmask, fm, ts, tm;
};

__device__ __forceinline__ BandFields band_fields(int mode, uint32_t words) {
    BandFields f;
    f.mul = kSlotMul << mode;
    f.wmask = (words - 1u) << 2;
    f.fm = mode == 0 ? 3u : mode == 1 ? 2u : 0u;
    f.tm = 4u << mode;
    f.ts = 29u - (uint32_t)mode;
    if (mode == 3) f.wmask &= ~4u;
    return f;
}

// Layout of an anchor's hashed slots (see slot_bits), the same for every lane:
// bits per counter, the largest counter, the largest key.
struct SlotLayout {
    uint32_t cb, ones, keys;
};
__device__ __forceinline__ SlotLayout slot_layout(uint32_t rank) {
    const uint32_t cb = slot_bits(rank);
    return SlotLayout{cb, (1u << cb) - 1u, ~0u >> (2u * cb)};
}

// Hashed counting: a slot holds the endpoint's key (anchor rank - endpoint
// rank, from 1) above two counters; an insert returns the counter's value
// before it, which is its share of C(x, 2).  A counter that passes its width
// is reported (`full`): the caller then counts the anchor in bands.
// LOCK: all of a lane's positions probe in lock step, so that their LDS round
// trips overlap (a slot, once claimed, keeps its key, so probing on meets the
// same slots in any order).  For the waves that share a table: 745 us instead
// of 1063 us on the heavier tier of the 20M-edge power-law graph.  The light
// waves have the LDS less loaded and keep the shorter code of one probe after
// the other: 433 us instead of 521 us there.
// lt: log2 of the slots in use, at least twice the wedges, so every probe ends.
template <int GP, bool LOCK>
__device__ __forceinline__ uint32_t hash_group(uint32_t* __restrict__ tab, const Group<GP>& g, uint32_t rx, int lt,
                                               const SlotLayout& sl, bool& full) {
    uint32_t key[GP], sh[GP], h[GP];
    uint32_t pend = 0;  // positions still probing
#pragma unroll
    for (int i = 0; i < GP; ++i) {
        key[i] = (rx - g.x[i]) & sl.keys;
        sh[i] = (uint32_t)((int32_t)(g.x[i] ^ g.tv[i]) >> 31) & sl.cb;
        h[i] = (key[i] * 0x9E3779B1u) >> (32 - lt);
        pend |= (i < g.nv ? 1u : 0u) << i;
    }
    uint32_t acc = 0;
    if constexpr (!LOCK) {
#pragma unroll
        for (int i = 0; i < GP; ++i) {
            if (!((pend >> i) & 1u)) continue;
            for (;;) {
                const uint32_t old = atomicCAS(&tab[h[i]], 0u, (key[i] << (2u * sl.cb)) | (1u << sh[i]));
                if (old == 0u) break;
                if ((old >> (2u * sl.cb)) == key[i]) {
                    const uint32_t c = (atomicAdd(&tab[h[i]], 1u << sh[i]) >> sh[i]) & sl.ones;
                    if (c == sl.ones) full = true;
                    acc += c;
                    break;
                }
                h[i] = (h[i] + 1u) & ((1u << lt) - 1u);
            }
        }
        return acc;
    }
    while (pend) {
        uint32_t old[GP], v[GP];
#pragma unroll
        for (int i = 0; i < GP; ++i) {
            old[i] = 0u;
            if ((pend >> i) & 1u) old[i] = atomicCAS(&tab[h[i]], 0u, (key[i] << (2u * sl.cb)) | (1u << sh[i]));
        }
#pragma unroll
        for (int i = 0; i < GP; ++i) {
            v[i] = 0u;
            if (old[i] != 0u && (old[i] >> (2u * sl.cb)) == key[i]) v[i] = atomicAdd(&tab[h[i]], 1u << sh[i]);
        }
        uint32_t next = 0;
#pragma unroll
        for (int i = 0; i < GP; ++i) {
            const bool other = old[i] != 0u && (old[i] >> (2u * sl.cb)) != key[i];
            next |= (other ? 1u : 0u) << i;
            h[i] = (h[i] + 1u) & ((1u << lt) - 1u);  // where another key was met
            const uint32_t c = (v[i] >> sh[i]) & sl.ones;
            if (c == sl.ones) full = true;
            acc += c;
        }
        pend &= next;
    }
    return acc;
}

// Per-vertex counts (FULL kernels).  A pair x, w with counters a and b holds
// C(a,2) + C(b,2) butterflies of x and of w, and each of its wedges is in one
// less than its counter's value of its middle's.  So once an anchor (or a band
// of it) is counted, its wedges are read again, the counter of each is looked
// up and what it gives its middle is summed per slice in LDS; then the
// counters give the endpoints' shares.  All in rank order; k_top_credit moves
// them to the ids.  Bound by the 64-bit atomics: on 2M power-law edges the
// walk kernels take 1.62 ms (the total alone 0.6 ms), 0.43 ms of it the
// endpoints' shares and 0.25 ms the second reading; the one-sided walk took
// 14.6 ms.

// The counters of key in the table.  It is there, so the search ends: in a
// simple graph no counter has carried into a key (a bound on the search, or an
// end at an empty slot, takes 40 to 50 us more on 2M power-law edges).
__device__ __forceinline__ uint32_t hash_look(const uint32_t* __restrict__ tab, uint32_t key, int lt,
                                              const SlotLayout& sl) {
    uint32_t h = (key * 0x9E3779B1u) >> (32 - lt);
    for (;;) {
        const uint32_t v = tab[h];
        if ((v >> (2u * sl.cb)) == key) return v;
        h = (h + 1u) & ((1u << lt) - 1u);
    }
}

// Adds what a wave's positions give to the words of their slices: v[i] to
// ys[at[i]], slices in order along the positions (GP per lane).  Neighbours
// mostly share a slice, and 64 lanes adding to one LDS word are served one by
// one, so the lanes that end in one slice are summed first.
template <int GP>
__device__ __forceinline__ void slice_add(uint32_t* __restrict__ ys, const uint32_t (&at)[GP], const uint32_t (&v)[GP]) {
    uint32_t any = 0, tail = v[GP - 1];
#pragma unroll
    for (int i = 0; i < GP; ++i) any |= v[i];
    if (!__any(any != 0u)) return;
    const uint32_t own = at[GP - 1];
#pragma unroll
    for (int i = 0; i < GP - 1; ++i) {
        if (at[i] == own) tail += v[i];
        else if (v[i]) atomicAdd(&ys[at[i]], v[i]);
    }
    const int lane = lane_id();
    const uint32_t sum = wave_inclusive_sum_dpp(tail);
    const uint32_t prev = (uint32_t)__shfl_up((int)own, 1, kWave);
    const unsigned long long heads = __ballot(lane == 0 || prev != own);
    const int h = 63 - __clzll(heads & (~0ull >> (63 - lane)));  // first lane of this lane's run
    const uint32_t before = (uint32_t)__shfl((int)sum, h > 0 ? h - 1 : 0, kWave);
    const bool last = lane == kWave - 1 || ((heads >> (lane + 1)) & 1ull);
    const uint32_t run = sum - (h > 0 ? before : 0u);
    if (last && run) atomicAdd(&ys[own], run);
}

// Second reading of one chunk's slices: what its wedges give the middles, per
// slice in ys (one word per lane, zero before and after), added to pv at y
// (this lane's middle).  At most 62 per wedge and 2^14 wedges.
template <int GP>
__device__ __forceinline__ void hash_credit(Flat f, uint32_t* __restrict__ mark, const uint32_t* __restrict__ stab,
                                            const uint32_t* __restrict__ ent, const uint32_t* __restrict__ tab, uint32_t rx,
                                            int lt, const SlotLayout& sl, uint32_t* __restrict__ ys,
                                            unsigned long long* __restrict__ pv, uint32_t y) {
    const int lane = lane_id();
    f.carry = 0;
    for (int32_t j0 = 0; j0 < f.total; j0 += GP * kWave) {
        Group<GP> g;
        flat_load<GP>(f, mark, stab, ent, j0, g);
        uint32_t give[GP];
#pragma unroll
        for (int i = 0; i < GP; ++i) {
            give[i] = 0;
            if (i >= g.nv) continue;
            const uint32_t v = hash_look(tab, (rx - g.x[i]) & sl.keys, lt, sl);
            give[i] = ((v >> ((uint32_t)((int32_t)(g.x[i] ^ g.tv[i]) >> 31) & sl.cb)) & sl.ones) - 1u;
        }
        slice_add<GP>(ys, g.sl, give);
    }
    __builtin_amdgcn_wave_barrier();
    const uint32_t v = ys[lane];
    if (v) {
        atomicAdd(&pv[y], (unsigned long long)v);
        ys[lane] = 0;
    }
    __builtin_amdgcn_wave_barrier();
}

// Endpoints' shares of slot v of a table (anchor rank rx, first vertex of its
// side xb).
__device__ __forceinline__ void hash_share(uint32_t v, uint32_t rx, uint32_t xb, const SlotLayout& sl,
                                           unsigned long long* __restrict__ pv) {
    const uint32_t a = v & sl.ones, b = (v >> sl.cb) & sl.ones, key = v >> (2u * sl.cb);
    const uint32_t s = a * (a - (a > 0u)) + b * (b - (b > 0u));
    if (s && key <= rx) atomicAdd(&pv[xb + rx - key], (unsigned long long)(s >> 1));
}

// A middle as read ahead: entry, end of its wedges, start of its list.
struct Mid {
    uint32_t e, cr, ms;
};

// First position in [lo, hi) of a rank-sorted list with rank >= r.
__device__ __forceinline__ uint32_t list_seek(const uint32_t* __restrict__ ent, uint32_t lo, uint32_t hi, uint32_t r) {
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (top_rank(ent[mid]) < r) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// The ranks of a band [lo, hi) below an anchor; first / last: it starts at the
// side's first rank / ends at the anchor.
struct TopRange {
    uint32_t lo, hi;
    bool first, last;
};

// Sum of squares of every counter of the band (its words only), cleared.
template <int MODE, int WG>
__device__ __forceinline__ unsigned long long reduce_words(uint32_t* __restrict__ cnt, uint32_t words) {
    PairSum<MODE, true> ps;
    for (uint32_t w4 = threadIdx.x; w4 < words / 4u; w4 += WG) {
        uint4* p = reinterpret_cast<uint4*>(&cnt[w4 * 4u]);
        const uint4 v = *p;
        if (v.x | v.y | v.z | v.w) {
            *p = uint4{0u, 0u, 0u, 0u};
            ps.add(v.x);
            ps.add(v.y);
            ps.add(v.z);
            ps.add(v.w);
        }
    }
    return ps.take();
}

__device__ __forceinline__ TopRange make_range(const TopBands& B, int32_t b, int32_t nbx, int32_t r) {
    TopRange rg;
    rg.first = b == 0;
    rg.last = b + 1 >= nbx;
    rg.lo = (uint32_t)band_lo(B, b);
    rg.hi = rg.last ? (uint32_t)r : (uint32_t)band_lo(B, b + 1);
    return rg;
}

// An anchor's place in its side: bands, rank, bands below it, list range.
struct TopAnchor {
    TopBands B;
    uint32_t a0, k;
    int32_t r, nbx;
};

__device__ __forceinline__ TopAnchor top_anchor(const TopArgs& a, uint32_t x) {
    TopAnchor t;
    const int side = x >= (uint32_t)a.n_u;
    t.B = a.bands[side];
    t.r = (int32_t)(side ? x - (uint32_t)a.n_u : x);
    t.nbx = t.r > 0 ? band_of(t.B, t.r - 1) + 1 : 0;
    t.a0 = a.off[x];
    t.k = a.kx[x];
    return t;
}

// Adds the workgroup's sum of acc to the total.
template <int WG, class Shared>
__device__ __forceinline__ void add_total(const TopArgs& a, Shared& sh, unsigned long long acc,
                                          unsigned long long bands) {
    acc = block_sum<WG>(acc, sh.red);
    if (threadIdx.x == 0 && acc) atomicAdd(&my_sums(a.st)->total, acc);
    if (threadIdx.x == 0 && bands) atomicAdd(&my_sums(a.st)->bands, bands);
}

// ------------------------------------------------------------------ bands
//
// One band of one of the heaviest anchors per task.  A hub's middles are
// mostly vertices of low degree whose slice of a band holds a few entries or
// none, so what bounds a band is the latency of reading the middles, not the
// wedges: a lane takes two consecutive middles there, and the first chunk of
// the next task is read while the current band is reduced.  The highest
// middles, whose slices hold thousands, go first and in small chunks, so that
// no wave is left alone with one.

// Middles per lane in the chunks of the lowest ones.
constexpr int kLaneMids = 2;

// Chunk layout: places from the top, in three sections of chunks of `size`
// middles (at most 64, a middle per lane), then chunks of kLaneMids per lane.
// Anchors of many wedges split their highest middles, whose slices of one band
// hold thousands each, further.
struct ChunkLayout {
    uint32_t c1, c2, c3;     // first chunk of sections 1, 2 and of the rest
    uint32_t s0, s1, s2;     // middles per chunk
};
__device__ __forceinline__ ChunkLayout chunk_layout(bool fine) {
    return fine ? ChunkLayout{32, 64, 80, 2, 8, 64} : ChunkLayout{16, 16, 32, 16, 16, 64};
}
constexpr unsigned long long kFineWork = 1ull << 18;
__device__ __forceinline__ uint32_t quad_chunks(const ChunkLayout& l, uint32_t k) {
    const uint32_t e0 = l.c1 * l.s0, e1 = e0 + (l.c2 - l.c1) * l.s1, e2 = e1 + (l.c3 - l.c2) * l.s2;
    if (k <= e0) return (k + l.s0 - 1u) / l.s0;
    if (k <= e1) return l.c1 + (k - e0 + l.s1 - 1u) / l.s1;
    if (k <= e2) return l.c2 + (k - e1 + l.s2 - 1u) / l.s2;
    return l.c3 + (k - e2 + kLaneMids * kWave - 1u) / (kLaneMids * kWave);
}

// Up to kLaneMids middles of a lane as read ahead: entry, end of the wedges,
// start of the list, index row (kNoIndex without one) and, once the row has
// been read, its two bounds for the band (the first one in place of the row).
struct Quad {
    uint32_t e[kLaneMids], cr[kLaneMids], ms[kLaneMids], i0[kLaneMids], i1[kLaneMids];
};

__device__ __forceinline__ void load_mids(uint32_t (&d)[kLaneMids], const uint32_t* __restrict__ src) {
    __builtin_memcpy(d, src, sizeof d);
}

// Reads chunk c of an anchor's k middles at a0 (c at or past the last chunk:
// none).  A slot without a middle gets an empty slice (end = start = 0).
__device__ __forceinline__ void quad_load(Quad& q, const TopArgs& a, uint32_t a0, uint32_t k, uint32_t n_ch,
                                          uint32_t c, const ChunkLayout& l) {
    const uint32_t lane = (uint32_t)lane_id();
#pragma unroll
    for (int j = 0; j < kLaneMids; ++j) {
        q.e[j] = q.cr[j] = q.ms[j] = 0;
        q.i0[j] = kNoIndex;
    }
    if (c >= n_ch) return;
    const uint32_t e0 = l.c1 * l.s0, e1 = e0 + (l.c2 - l.c1) * l.s1, e2 = e1 + (l.c3 - l.c2) * l.s2;
    if (c < l.c3) {  // one middle per lane
        const uint32_t size = c < l.c1 ? l.s0 : c < l.c2 ? l.s1 : l.s2;
        const uint32_t first = c < l.c1 ? c * l.s0 : c < l.c2 ? e0 + (c - l.c1) * l.s1 : e1 + (c - l.c2) * l.s2;
        const uint32_t i = first + lane;
        if (lane < size && i < k) {
            const uint32_t p = a0 + (k - 1u - i);
            q.e[0] = a.ent[p];
            q.cr[0] = a.cross[p];
            q.ms[0] = a.mstart[p];
            q.i0[0] = a.mbase[p];
        }
    } else {  // places i .. i + kLaneMids - 1 from the top, in memory order (k > e2 >= kLaneMids)
        const uint32_t i = e2 + (c - l.c3) * (kLaneMids * kWave) + kLaneMids * lane;
        if (i < k) {
            const uint32_t hi = k - 1u - i;  // the highest of the lane's middles
            const uint32_t lo = hi >= kLaneMids - 1u ? hi - (kLaneMids - 1u) : 0u;
            const uint32_t p = a0 + lo;
            load_mids(q.e, a.ent + p);
            load_mids(q.cr, a.cross + p);
            load_mids(q.ms, a.mstart + p);
            load_mids(q.i0, a.mbase + p);
#pragma unroll
            for (int j = 0; j < kLaneMids; ++j)
                if (lo + (uint32_t)j > hi) {
                    q.cr[j] = q.ms[j] = 0;
                    q.i0[j] = kNoIndex;
                }
        }
    }
}

__device__ __forceinline__ void quad_bounds(Quad& q, const TopArgs& a, int32_t b) {
#pragma unroll
    for (int j = 0; j < kLaneMids; ++j) {
        q.i1[j] = 0;
        if (q.i0[j] != kNoIndex) {
            uint32_t d[2];
            __builtin_memcpy(d, a.idx + q.i0[j] + (uint32_t)b, 8);
            q.i0[j] = d[0];
            q.i1[j] = d[1];
        }
    }
}

constexpr int kQuadGP = 4;
// LDS of one wave: a 16-bit mark per position of a group, a word per slice.
struct QuadLds {
    alignas(16) uint32_t tab[kLaneMids * kWave];
    alignas(16) uint32_t mark[kQuadGP * kWave / 2];
};
typedef uint16_t __attribute__((may_alias)) mark16;

// A task: the anchor's list range and rank, and the band.
struct TopTask {
    uint32_t a0, k, r, lo, hi, words;
    int32_t b, mode;
    uint32_t x;  // the anchor
    uint32_t flags;  // bit 0: the band is the side's first; bit 1: the anchor lies in it; bit 2: fine chunks
};

// A task read from LDS, in scalar registers.
__device__ __forceinline__ TopTask uniform_task(const TopTask& s) {
    auto u = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); };
    return TopTask{u(s.a0),         u(s.k),           u(s.r),          u(s.lo),        u(s.hi), u(s.words),
                   (int32_t)u((uint32_t)s.b), (int32_t)u((uint32_t)s.mode), u(s.x), u(s.flags)};
}

template <int WG, int BW, bool FULL>
struct BandShared {
    alignas(16) uint32_t cnt[BW];
    QuadLds flat[WG / kWave];
    uint32_t ys[FULL ? WG / kWave : 1][FULL ? kLaneMids * kWave : 1];  // per slice: what its wedges give the middle
    unsigned long long red[WG / kWave];
    TopTask task[2];
    uint32_t next;  // next chunk of middles
};

// The slices of a wave's lanes, laid end to end.
struct QuadFlat {
    int32_t total, ex, len[kLaneMids];
    uint32_t carry;
    bool quad;  // more than one slice per lane
};

__device__ __forceinline__ void quad_begin(QuadFlat& f, QuadLds& sh, const Quad& q, const TopArgs& a,
                                           const TopTask& t, bool quad) {
    const bool first = t.flags & 1u, last = t.flags & 2u;
    uint32_t st[kLaneMids];
    int32_t sum = 0;
    auto slice = [&](int j) {
        uint32_t s, e;
        if (q.i0[j] != kNoIndex) {
            s = first ? q.ms[j] : min(q.i0[j], q.cr[j]);
            e = last ? q.cr[j] : min(q.i1[j], q.cr[j]);
        } else {  // a short list: searched
            s = first ? q.ms[j] : list_seek(a.ent, q.ms[j], q.cr[j], t.lo);
            e = last ? q.cr[j] : list_seek(a.ent, s, q.cr[j], t.hi);
        }
        st[j] = s;
        f.len[j] = (int32_t)(e - s);
        sum += f.len[j];
    };
    slice(0);
    if (quad) {
#pragma unroll
        for (int j = 1; j < kLaneMids; ++j) slice(j);
    } else {
#pragma unroll
        for (int j = 1; j < kLaneMids; ++j) {
            st[j] = 0;
            f.len[j] = 0;
        }
    }
    const int32_t inc = (int32_t)wave_inclusive_sum_dpp((uint32_t)sum);
    f.total = __builtin_amdgcn_readlane(inc, kWave - 1);
    f.ex = inc - sum;
    f.carry = 0;
    f.quad = quad;
    int32_t ex = f.ex;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < kLaneMids; ++j) {
        sh.tab[kLaneMids * lane_id() + j] = ((st[j] - (uint32_t)ex) & 0x3fffffffu) | (q.e[j] & 0x80000000u);
        ex += f.len[j];
    }
    __builtin_amdgcn_wave_barrier();
}

// Slice words of the group at position j0 (groups in order) of a chunk with
// wedges, several slices per lane (16-bit marks); see flat_load.
__device__ __forceinline__ void quad_words(QuadFlat& f, QuadLds& sh, int32_t j0, uint32_t (&tv)[kQuadGP],
                                           uint32_t (&at)[kQuadGP]) {
    constexpr int GP = kQuadGP;
    const int lane = lane_id();
    // marks hold the byte offset of the slice's word, plus 4
    mark16* const mark = reinterpret_cast<mark16*>(sh.mark);
    int32_t d = f.ex - j0;
    if (f.len[0] > 0 && (uint32_t)d < (uint32_t)(GP * kWave)) mark[d] = (mark16)(4 * kLaneMids * lane + 4);
    if (f.quad) {
#pragma unroll
        for (int j = 1; j < kLaneMids; ++j) {
            d += f.len[j - 1];
            if (f.len[j] > 0 && (uint32_t)d < (uint32_t)(GP * kWave))
                mark[d] = (mark16)(4 * kLaneMids * lane + 4 * j + 4);
        }
    }
    __builtin_amdgcn_wave_barrier();
    static_assert(GP == 4, "a lane's marks are one 8-byte word");
    const uint2 w = reinterpret_cast<const uint2*>(sh.mark)[lane];
    reinterpret_cast<uint2*>(sh.mark)[lane] = uint2{0u, 0u};
    __builtin_amdgcn_wave_barrier();
    uint32_t k[GP] = {w.x & 0xffffu, w.x >> 16, w.y & 0xffffu, w.y >> 16};
#pragma unroll
    for (int i = 1; i < GP; ++i) k[i] = max(k[i], k[i - 1]);
    const uint32_t inc = wave_inclusive_max_dpp(k[GP - 1]);
    const uint32_t before =
        max((uint32_t)__builtin_amdgcn_update_dpp(0, (int)inc, 0x138, 0xf, 0xf, false), f.carry);
    f.carry = max(f.carry, (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1));
    // every k is at least 4: position 0 is marked
#pragma unroll
    for (int i = 0; i < GP; ++i) {
        at[i] = max(k[i], before) - 4u;  // byte offset of the slice's word
        tv[i] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(sh.tab) + at[i]);
    }
}

// Counts the task's wedges (all waves).  cur holds the wave's first chunk,
// read ahead.  Returns minus the wedges counted (lane 0 of each wave).
//
// One group is in flight at any time: while it is, the next group's slice
// words are worked out (a chain of LDS round trips, or the next chunk's
// layout); then the group in flight is turned into counter fields, the next
// group's loads go out, and only then are the fields added.  One copy of each
// step keeps the loop inside the registers and the instruction cache (two
// groups by turns, with every step twice and another copy for 32-bit counters,
// spilled and took 9.95 ms instead of 6.7 ms on the 20M-edge power-law graph).
template <int WG, int BW, bool FULL>
__device__ __forceinline__ unsigned long long band_walk(BandShared<WG, BW, FULL>& sh, const TopArgs& a,
                                                        const TopTask& t, Quad& cur) {
    constexpr int GP = kQuadGP;
    const int lane = lane_id();
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    QuadLds& fl = sh.flat[wave];
    const BandFields bf = band_fields(t.mode, t.words);
    const bool wide = t.mode == 3;
    const ChunkLayout l = chunk_layout(t.flags & 4u);
    const uint32_t n_ch = quad_chunks(l, t.k);
    uint32_t c = WG / kWave - 1u - wave;  // wave 0, which takes the tasks, gets the lightest chunk
    unsigned long long acc = 0;
    QuadFlat f;
    f.total = f.ex = 0;
    f.carry = 0;
    f.quad = false;
    // cur: 0 = the next chunk, ready; 1 = its index rows are still to be read;
    // 2 = all of it
    int stage = 0;
    auto read_on = [&]() {  // one stage of reading the next chunk ahead
        if (stage == 2) {
            uint32_t q = 0;
            if (lane == 0) q = atomicAdd(&sh.next, 1u);  // starts at the number of waves
            c = (uint32_t)__builtin_amdgcn_readfirstlane((int)q);
            quad_load(cur, a, t.a0, t.k, n_ch, c, l);
            stage = 1;
        } else if (stage == 1) {
            quad_bounds(cur, a, t.b);
            stage = 0;
        }
    };
    const char* const ent = reinterpret_cast<const char*>(a.ent);
    char* const cnt = reinterpret_cast<char*>(sh.cnt);
    uint32_t x[GP], tv[GP];  // the group in flight
    int32_t nv = 0;          // this lane's positions of it holding wedges
    bool full = false, have = false;
    for (int32_t j0 = 0;; j0 += GP * kWave) {
        if (j0 >= f.total) {  // the next chunk with wedges in the band
            j0 = 0;
            f.total = 0;
            while (c < n_ch) {
                while (stage) read_on();
                if (c >= n_ch) break;
                quad_begin(f, fl, cur, a, t, c >= l.c3);
                stage = 2;
                if (f.total > 0) break;
            }
            if (lane == 0) acc -= (unsigned long long)f.total;
        }
        const bool more = f.total > 0;
        uint32_t tn[GP], at[GP];
        if (more) quad_words(f, fl, j0, tn, at);
        __builtin_amdgcn_sched_barrier(0);
        uint32_t byte[GP], inc[GP];
#pragma unroll
        for (int i = 0; i < GP; ++i) {
            // the multiply reads the low 24 bits: the sign on top does not matter
            const uint32_t p = mul_u24(x[i], bf.mul), ty = x[i] ^ tv[i];  // type in bit 31
            byte[i] = p & bf.wmask;
            inc[i] = 1u << ((((p & bf.fm) << 3) | ((ty >> bf.ts) & bf.tm)) & 31u);
            if (wide) {
                byte[i] |= ty >> 31 << 2;
                inc[i] = 1u;
            }
        }
        const bool had = have, all = full;
        const int32_t n = nv;
        __builtin_amdgcn_sched_barrier(0);
        if (more) {
            const int32_t j = j0 + lane * GP;
            nv = f.total - j;
            full = j0 + GP * kWave <= f.total;
            uint32_t off[GP];  // byte offsets: the shift drops the sign
#pragma unroll
            for (int i = 0; i < GP; ++i) off[i] = (tn[i] + (uint32_t)(j + i)) << 2;
            if (!full) {
#pragma unroll
                for (int i = 0; i < GP; ++i) off[i] = i < nv ? off[i] : 0u;
            }
#pragma unroll
            for (int i = 0; i < GP; ++i) {
                tv[i] = tn[i];
                x[i] = *reinterpret_cast<const uint32_t*>(ent + off[i]);
            }
        }
        have = more;
        __builtin_amdgcn_sched_barrier(0);
        if (had && all) {
#pragma unroll
            for (int i = 0; i < GP; ++i)
                (void)__hip_atomic_fetch_add(reinterpret_cast<uint32_t*>(cnt + byte[i]), inc[i], __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_WORKGROUP);
        } else if (had) {
#pragma unroll
            for (int i = 0; i < GP; ++i)
                if (i < n)
                    (void)__hip_atomic_fetch_add(reinterpret_cast<uint32_t*>(cnt + byte[i]), inc[i], __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if (!more) break;
        if (c < n_ch && stage) read_on();
    }
    return acc;
}

// The second reading of a counted band's wedges (FULL): chunks are dealt as in
// band_walk; the middles' shares are summed per slice, 32 bits wide (a band of
// 32-bit counters, whose sums may need more, adds each share at once; its ys
// hold the slices' middles).
template <int WG, int BW>
__device__ __forceinline__ void band_credit(BandShared<WG, BW, true>& sh, const TopArgs& a, const TopTask& t) {
    constexpr int GP = kQuadGP;
    const int lane = lane_id();
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    QuadLds& fl = sh.flat[wave];
    uint32_t* const ys = sh.ys[wave];
    const BandFields bf = band_fields(t.mode, t.words);
    const bool wide = t.mode == 3;
    const uint32_t ones = wide ? ~0u : (1u << (4 << t.mode)) - 1u;
    const ChunkLayout l = chunk_layout(t.flags & 4u);
    const uint32_t n_ch = quad_chunks(l, t.k);
    const uint32_t yb = t.x < (uint32_t)a.n_u ? (uint32_t)a.n_u : 0u;
    const char* const ent = reinterpret_cast<const char*>(a.ent);
    const char* const cnt = reinterpret_cast<const char*>(sh.cnt);
    uint32_t c = WG / kWave - 1u - wave;
    Quad q;
    quad_load(q, a, t.a0, t.k, n_ch, c, l);
    while (c < n_ch) {
        quad_bounds(q, a, t.b);
        QuadFlat f;
        quad_begin(f, fl, q, a, t, c >= l.c3);
        uint32_t y[kLaneMids];
#pragma unroll
        for (int j = 0; j < kLaneMids; ++j) {
            y[j] = yb + top_rank(q.e[j]);
            if (wide) ys[kLaneMids * lane + j] = y[j];
        }
        __builtin_amdgcn_wave_barrier();
        uint32_t next = 0;
        if (lane == 0) next = atomicAdd(&sh.next, 1u);
        c = (uint32_t)__builtin_amdgcn_readfirstlane((int)next);
        quad_load(q, a, t.a0, t.k, n_ch, c, l);  // ahead
        for (int32_t j0 = 0; j0 < f.total; j0 += GP * kWave) {
            uint32_t tv[GP], at[GP], x[GP];
            quad_words(f, fl, j0, tv, at);
            const int32_t j = j0 + lane * GP, nv = f.total - j;
#pragma unroll
            for (int i = 0; i < GP; ++i)
                x[i] = *reinterpret_cast<const uint32_t*>(ent + (i < nv ? (tv[i] + (uint32_t)(j + i)) << 2 : 0u));
            uint32_t give[GP];
#pragma unroll
            for (int i = 0; i < GP; ++i) {
                at[i] >>= 2;
                give[i] = 0;
                if (i >= nv) continue;
                const uint32_t p = mul_u24(x[i], bf.mul), ty = x[i] ^ tv[i];
                const uint32_t word = (p & bf.wmask) | (wide ? ty >> 31 << 2 : 0u);
                const uint32_t sh_ = wide ? 0u : (((p & bf.fm) << 3) | ((ty >> bf.ts) & bf.tm)) & 31u;
                const uint32_t v = (*reinterpret_cast<const uint32_t*>(cnt + word) >> sh_) & ones;
                if (!wide) give[i] = v - 1u;
                else if (v > 1u) atomicAdd(&a.pv[ys[at[i]]], (unsigned long long)(v - 1u));
            }
            slice_add<GP>(ys, at, give);
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < kLaneMids; ++j) {
            const uint32_t v = ys[kLaneMids * lane + j];
            if (v) {
                if (!wide) atomicAdd(&a.pv[y[j]], (unsigned long long)v);
                ys[kLaneMids * lane + j] = 0;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Endpoints' shares of a counted band, which is cleared; returns this thread's
// sum.  Slot s of the band holds the rank r in it with r kSlotMul = s modulo
// the band's slots; no other slot holds anything.
template <int WG>
__device__ __forceinline__ unsigned long long share_words(uint32_t* __restrict__ cnt, const TopArgs& a,
                                                          const TopTask& t) {
    unsigned long long sum = 0;
    const uint32_t xb = t.x < (uint32_t)a.n_u ? 0u : (uint32_t)a.n_u;
    auto give = [&](uint32_t slot, uint32_t slots, unsigned long long ca, unsigned long long cb) {
        const unsigned long long s = (ca * (ca - (ca > 0)) + cb * (cb - (cb > 0))) / 2ull;
        if (!s) return;
        const uint32_t r = t.lo + ((slot * kSlotInv - t.lo) & (slots - 1u));
        if (r >= t.hi) return;
        atomicAdd(&a.pv[xb + r], s);
        sum += s;
    };
    if (t.mode == 3) {
        uint2* p = reinterpret_cast<uint2*>(cnt);
        for (uint32_t i = threadIdx.x; i < t.words / 2u; i += WG) {
            const uint2 v = p[i];
            if (v.x | v.y) {
                p[i] = uint2{0u, 0u};
                give(i, t.words / 2u, v.x, v.y);
            }
        }
        return sum;
    }
    // a and b of an endpoint sum to at most 65535 here: 32 bits hold the shares
    const uint32_t per = 4u >> t.mode, bits = 4u << t.mode, ones = (1u << bits) - 1u;  // slots per word, counter bits
    const uint32_t slots = t.words * per;
    const uint32_t pairs = t.mode == 0 ? 0xeeeeeeeeu : t.mode == 1 ? 0xfefefefeu : 0xfffefffeu;  // a counter of 2 or more
    auto word = [&](uint32_t i, uint32_t v) {
        if (!(v & pairs)) return;
        for (uint32_t k = 0; k < per; ++k, v = bits == 16u ? 0u : v >> (2u * bits)) {
            const uint32_t ca = v & ones, cb = (v >> bits) & ones;
            const uint32_t s = (ca * (ca - (ca > 0u)) >> 1) + (cb * (cb - (cb > 0u)) >> 1);
            if (!s) continue;
            const uint32_t r = t.lo + (((i * per + k) * kSlotInv - t.lo) & (slots - 1u));
            if (r >= t.hi) continue;
            atomicAdd(&a.pv[xb + r], (unsigned long long)s);
            sum += s;
        }
    };
    for (uint32_t w4 = threadIdx.x; w4 < t.words / 4u; w4 += WG) {
        uint4* p = reinterpret_cast<uint4*>(&cnt[w4 * 4u]);
        const uint4 v = *p;
        if (!(v.x | v.y | v.z | v.w)) continue;
        *p = uint4{0u, 0u, 0u, 0u};
        word(w4 * 4u, v.x);
        word(w4 * 4u + 1u, v.y);
        word(w4 * 4u + 2u, v.z);
        word(w4 * 4u + 3u, v.w);
    }
    return sum;
}

// Bound by reading the middles: every band of an anchor reads the same middles
// (16 bytes each) and neighbouring words of their index rows.  From kXcdAnchors
// anchors on, the bands of one anchor are therefore tasks of one XCD, one after
// the other, which find them in its L2: 31.2 -> 26.3 GB read per 20M-edge
// power-law count (at about 5 TB/s) and 9.85 -> 9.09 ms for the call, against
// one queue band by band.
constexpr uint32_t kXcdAnchors = 512;
template <int WG, int BW, bool FULL>
__global__ __launch_bounds__(WG, 4) void k_top_bands(TopArgs a) {
    if (*(volatile const int32_t*)&a.st->flags) return;  // input error: nothing to count
    const uint32_t n_split = *(volatile const uint32_t*)&a.tc->n_tier[0];
    const uint32_t n_all = n_split + *(volatile const uint32_t*)&a.tc->n_extra;
    const uint32_t nb_max = *(volatile const uint32_t*)&a.tc->nb_max;
    // Queue v of eight holds the anchors v, v + 8, ..., each with its bands one
    // after the other; workgroup b starts in queue b % 8 (its XCD).  A single
    // queue (few anchors) goes band by band.
    const uint32_t nq = n_all >= kXcdAnchors ? 8u : 1u;
    auto length = [&](uint32_t v) { return (unsigned long long)((n_all - v + nq - 1u) / nq) * nb_max; };
    auto groups = [&](uint32_t v) { return (gridDim.x - v + nq - 1u) / nq; };  // workgroups that start there
    uint32_t queue = blockIdx.x % nq;
    unsigned long long ahead = blockIdx.x / nq;
    if (n_all == 0 || ahead >= length(queue)) return;  // idle ones touch no queue
    __shared__ BandShared<WG, BW, FULL> sh;
    const int tid = threadIdx.x, lane = lane_id();
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid / kWave));
    for (int i = tid; i < BW; i += WG) sh.cnt[i] = 0;
    reinterpret_cast<uint2*>(sh.flat[wave].mark)[lane] = uint2{0u, 0u};
    if constexpr (FULL)
        for (int j = lane; j < kLaneMids * kWave; j += kWave) sh.ys[wave][j] = 0;
    // Thread 0 takes the next task that has a band (widest counters, which
    // hold most wedges, first), each pop sent out one task ahead; an empty
    // queue gives way to the next one; k = 0 marks the end.
    uint32_t tried = 1;
    auto take = [&](TopTask& t) {
        for (;;) {
            t.k = 0;
            while (ahead >= length(queue)) {
                if (a.statik || tried == nq) return;
                ++tried;
                queue = queue + 1u == nq ? 0u : queue + 1u;
                ahead = groups(queue) + atomicAdd(&a.tc->queue[queue], 1ull);
            }
            const unsigned long long i = ahead;
            const uint32_t own = queue;
            ahead = a.statik ? i + groups(own) : groups(own) + atomicAdd(&a.tc->queue[own], 1ull);
            const uint32_t q = nq == 1u ? (uint32_t)(i % n_all) : own + nq * (uint32_t)(i / nb_max);
            const uint32_t id = q < n_split ? a.order[q] : a.extra[q - n_split];
            const TopAnchor x = top_anchor(a, id);
            const int32_t b = (int32_t)(nb_max - 1u - (uint32_t)(nq == 1u ? i / n_all : i % nb_max));
            if (b >= x.nbx) continue;
            const TopRange rg = make_range(x.B, b, x.nbx, x.r);
            t = TopTask{x.a0,  x.k, (uint32_t)x.r,         rg.lo, rg.hi, 1u << x.B.lw,
                        b,     band_mode(x.B, b), id, (rg.first ? 1u : 0u) | (rg.last ? 2u : 0u) | (a.work[id] >= kFineWork ? 4u : 0u)};
            return;
        }
    };
    if (tid == 0) {
        sh.next = WG / kWave;
        take(sh.task[0]);
    }
    __syncthreads();
    unsigned long long acc = 0, bands = 0;
    Quad cur;
    auto first_chunk = [&](const TopTask& t) {
        const ChunkLayout l = chunk_layout(t.flags & 4u);
        quad_load(cur, a, t.a0, t.k, quad_chunks(l, t.k), WG / kWave - 1u - wave, l);
    };
    {
        const TopTask t = uniform_task(sh.task[0]);
        if (t.k > 0) {
            first_chunk(t);
            quad_bounds(cur, a, t.b);
        }
    }
    for (uint32_t it = 0;; it ^= 1u) {
        const TopTask t = uniform_task(sh.task[it]);
        if (t.k == 0) break;
        if (tid == 0) take(sh.task[it ^ 1u]);
        unsigned long long mine = band_walk(sh, a, t, cur);
        __syncthreads();
        if constexpr (FULL) {
            if (tid == 0) sh.next = WG / kWave;
            __syncthreads();
            band_credit(sh, a, t);
            __syncthreads();
        }
        const TopTask n = uniform_task(sh.task[it ^ 1u]);
        if (n.k > 0) first_chunk(n);
        if (tid == 0) sh.next = WG / kWave;
        if constexpr (FULL) {
            const unsigned long long s = share_words<WG>(sh.cnt, a, t);
            const unsigned long long w = wave_sum(s);
            if (lane == 0 && w) atomicAdd(&a.pv[t.x], w);
            mine = 2ull * s;
        } else if (t.mode == 0) mine += reduce_words<0, WG>(sh.cnt, t.words);
        else if (t.mode == 1) mine += reduce_words<1, WG>(sh.cnt, t.words);
        else if (t.mode == 2) mine += reduce_words<2, WG>(sh.cnt, t.words);
        else mine += reduce_words<3, WG>(sh.cnt, t.words);
        if (n.k > 0) quad_bounds(cur, a, n.b);
        ++bands;
        acc += mine;
        __syncthreads();
    }
    add_total<WG>(a, sh, acc, bands);
}

// ------------------------------------------------------- hashed workgroups
//
// Anchors of the middle of the range: one anchor per task and workgroup, all
// its wedges in one hashed table of at least twice as many slots, so the cost
// follows the wedges and not the ranks below the anchor (in bands they held a
// few dozen wedges each), and slices need no index: a middle's wedges are its
// whole prefix.  Chunks of CH middles, highest first, go to the waves in turn;
// the next anchor is read while this one's table is cleared.  An anchor with a
// counter past its width is left to the bands (kernel k_top_bands runs after
// this one).
template <int WG, int LTMAX, bool FULL>
struct HashShared {
    alignas(16) uint32_t tab[1 << LTMAX];
    FlatLds<4> flat[WG / kWave];
    unsigned long long red[WG / kWave];
    TopTask task[2];
    uint32_t full, any;
    uint32_t ys[FULL ? WG / kWave : 1][FULL ? kWave : 1];
};

template <int WG, int LTMAX, int CH0, int CH, bool FULL>
__global__ __launch_bounds__(WG, 4) void k_top_hash(TopArgs a, int tier) {
    if (*(volatile const int32_t*)&a.st->flags) return;
    constexpr int NW = WG / kWave, GP = 4;
    const uint32_t p0 = *(volatile const uint32_t*)&a.tc->n_tier[tier];
    const uint32_t p1 = *(volatile const uint32_t*)&a.tc->n_tier[tier + 1];
    const uint32_t n_tasks = (p1 - p0 + (uint32_t)a.queue_chunk - 1u) / (uint32_t)a.queue_chunk;
    if (blockIdx.x >= n_tasks) return;  // the first task is the workgroup's own: idle ones touch no queue
    __shared__ HashShared<WG, LTMAX, FULL> sh;
    const int tid = threadIdx.x, lane = lane_id();
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid / kWave));
    FlatLds<GP>& fl = sh.flat[wave];
    for (int i = tid; i < (1 << LTMAX); i += WG) sh.tab[i] = 0;
    fl.mark[lane] = 0u;
    const uint32_t w0 = NW - 1u - wave;  // wave 0, which takes the tasks, gets the lightest chunks
    unsigned int* queue = &a.tc->queue_hash[tier];
    // Thread 0 takes queue_chunk anchors at a time, each pop sent out one
    // task ahead; k = 0 marks the end.
    unsigned long long at = 0, end = 0;
    uint32_t ahead = blockIdx.x;
    auto take = [&](TopTask& t) {
        if (at == end) {
            const uint32_t i = ahead;
            if (i < n_tasks) ahead = a.statik ? i + gridDim.x : gridDim.x + atomicAdd(queue, 1u);
            at = p0 + (unsigned long long)i * (uint32_t)a.queue_chunk;
            end = min(at + (uint32_t)a.queue_chunk, (unsigned long long)p1);
        }
        t.k = 0;
        if (at >= end) {
            end = at;
            return;
        }
        const uint32_t x = a.order[at++];
        t.a0 = a.off[x];
        t.r = x >= (uint32_t)a.n_u ? x - (uint32_t)a.n_u : x;
        t.lo = x;
        const uint32_t w = (uint32_t)a.work[x];  // below 2^(LTMAX - 1)
        t.mode = max(8, 33 - __clz((int)(w - 1u)));  // log2 of the slots: 2 w or more
        t.k = a.kx[x];
    };
    if (tid == 0) {
        sh.full = sh.any = 0;
        take(sh.task[0]);
    }
    if constexpr (FULL) sh.ys[wave][lane] = 0;
    // chunk c's middles from the highest down: CH0 each in the first NW chunks
    // (the longest lists), CH in the others; the other lanes read the
    // anchor's first entry and hold nothing
    auto mids = [&](const TopTask& t, uint32_t c, Mid& m, bool& has) {
        const uint32_t i = (c < NW ? c * CH0 : NW * CH0 + (c - NW) * CH) + (uint32_t)lane;
        has = lane < (c < NW ? CH0 : CH) && i < t.k;
        const uint32_t p = t.a0 + (has ? t.k - 1u - i : 0u);
        m.e = a.ent[p];
        m.cr = a.cross[p];
        m.ms = a.mstart[p];
    };
    auto clear = [&](int lt) {
        uint4* t4 = reinterpret_cast<uint4*>(sh.tab);
        for (int i = tid; i < (1 << lt) / 4; i += WG) t4[i] = uint4{0u, 0u, 0u, 0u};
    };
    __syncthreads();
    unsigned long long acc = 0;
    Mid m;
    bool has = false;
    {
        const TopTask t = uniform_task(sh.task[0]);
        if (t.k > 0) mids(t, w0, m, has);
    }
    for (uint32_t it = 0;; it ^= 1u) {
        const TopTask t = uniform_task(sh.task[it]);
        if (t.k == 0) break;
        if (tid == 0) take(sh.task[it ^ 1u]);
        const uint32_t n_ch = t.k <= NW * CH0 ? (t.k + CH0 - 1u) / CH0 : NW + (t.k - NW * CH0 + CH - 1u) / CH;
        const SlotLayout sl = slot_layout(t.r);
        uint32_t s = 0;
        bool full = false;
        for (uint32_t c = w0; c < n_ch; c += NW) {
            Flat f;
            flat_begin(f, fl.tab, m.ms, has ? (int32_t)(m.cr - m.ms) : 0, m.e);
            Group<GP> ga, gb;
            flat_load<GP>(f, fl.mark, fl.tab, a.ent, 0, ga);
            if (c + NW < n_ch) mids(t, c + NW, m, has);
            __builtin_amdgcn_sched_barrier(0);
            for (int32_t j0 = 0; j0 < f.total;) {  // two groups by turns, the next one in flight
                j0 += GP * kWave;
                if (j0 < f.total) flat_load<GP>(f, fl.mark, fl.tab, a.ent, j0, gb);
                __builtin_amdgcn_sched_barrier(0);
                s += hash_group<GP, true>(sh.tab, ga, t.r, t.mode, sl, full);
                if (j0 >= f.total) break;
                j0 += GP * kWave;
                if (j0 < f.total) flat_load<GP>(f, fl.mark, fl.tab, a.ent, j0, ga);
                __builtin_amdgcn_sched_barrier(0);
                s += hash_group<GP, true>(sh.tab, gb, t.r, t.mode, sl, full);
            }
        }
        if (full) sh.full = 1u;
        if (FULL && s) sh.any = 1u;
        __syncthreads();
        const bool bad = sh.full != 0;
        if constexpr (FULL) {
            if (!bad && sh.any) {  // the same for every thread
                const uint32_t yb = t.lo < (uint32_t)a.n_u ? (uint32_t)a.n_u : 0u;
                for (uint32_t c = w0; c < n_ch; c += NW) {
                    mids(t, c, m, has);
                    Flat f;
                    flat_begin(f, fl.tab, m.ms, has ? (int32_t)(m.cr - m.ms) : 0, m.e);
                    hash_credit<GP>(f, fl.mark, fl.tab, a.ent, sh.tab, t.r, t.mode, sl, sh.ys[wave], a.pv,
                                    yb + top_rank(m.e));
                }
                const unsigned long long w = wave_sum((unsigned long long)s);
                if (lane == 0 && w) atomicAdd(&a.pv[t.lo], w);
                __syncthreads();
                if (tid == 0) sh.any = 0;
                for (int i = tid; i < (1 << t.mode); i += WG) {
                    const uint32_t v = sh.tab[i];
                    if (v) hash_share(v, t.r, (uint32_t)a.n_u - yb, sl, a.pv);
                }
                __syncthreads();
            }
        }
        const TopTask n = uniform_task(sh.task[it ^ 1u]);
        if (n.k > 0) mids(n, w0, m, has);
        unsigned long long mine = bad ? 0ull : 2ull * s;
        if (bad && tid == 0) a.extra[atomicAdd(&a.tc->n_extra, 1u)] = t.lo;
        clear(t.mode);
        acc += mine;
        __syncthreads();
        if (bad) {  // the same for every thread
            if (tid == 0) sh.full = 0;
            __syncthreads();
        }
    }
    add_total<WG>(a, sh, acc, 0);
}

// ------------------------------------------------------------ wave regime
//
// Light anchors (at most kLightMaxWork wedges; at most 63 middles, see
// k_top_schedule): one wave each, a
// hashed table of 2048 slots per wave, no barrier.  The wave reads ahead: an
// anchor's place in the schedule three anchors before it is counted, its list
// range two before, its middles one before, and its first group of endpoints
// before the previous one's inserts.
constexpr int kTopLightWG = 256, kTopLightLT = 11, kLightGP = 4;
static_assert((1 << kTopLightLT) >= 2 * kLightMaxWork, "the table stays at most half full");

// A light anchor read ahead: vertex and list range.
struct LightHead {
    uint32_t x, a0, k;
};

template <bool FULL>
__global__ __launch_bounds__(kTopLightWG, 4) void k_top_light(TopArgs a) {
    if (*(volatile const int32_t*)&a.st->flags) return;
    constexpr int NW = kTopLightWG / kWave, TW = 1 << kTopLightLT, GP = kLightGP;
    __shared__ alignas(16) uint32_t tabs[NW][TW];
    __shared__ unsigned long long red[NW];
    __shared__ FlatLds<GP> flat[NW][2];  // two slice tables, alternating; the first one's marks serve both
    const int lane = lane_id();
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    uint32_t* tab = tabs[wave];
    uint32_t* mark = flat[wave][0].mark;
    auto clear = [&](int words) {
        uint4* t4 = reinterpret_cast<uint4*>(tab);
        for (int i = lane; i < words / 4; i += kWave) t4[i] = uint4{0u, 0u, 0u, 0u};
        __builtin_amdgcn_wave_barrier();
    };
    clear(TW);
    mark[lane] = 0u;
    __shared__ uint32_t ys[FULL ? NW : 1][FULL ? kWave : 1];
    if constexpr (FULL) ys[wave][lane] = 0u;
    __builtin_amdgcn_wave_barrier();
    const uint32_t n_heavy = *(volatile const uint32_t*)&a.tc->n_tier[kTopTiers];
    const uint32_t n_walk = *(volatile const uint32_t*)&a.tc->n_walk;
    // a fixed deal: the anchors' work is bounded and they are listed by rank,
    // so chunks at equal distances are alike (a queue cost more than it evened
    // out: every pop is an atomic on one address)
    const uint32_t n_light = n_walk > n_heavy ? n_walk - n_heavy : 0u;  // none: n_walk is 0
    const uint32_t n_waves = gridDim.x * NW;
    const uint32_t lc = max(1u, min((uint32_t)a.light_chunk, n_light / (n_waves * 4u)));
    const uint32_t n_tasks = (n_light + lc - 1) / lc;
    // A zero the compiler cannot see keeps the reads ahead on the vector
    // path: scalar loads share their counter with LDS operations and return
    // out of order, so the next LDS use would wait for them.
    uint32_t zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
    unsigned long long acc = 0;
    for (uint32_t task = blockIdx.x * NW + wave; task < n_tasks; task += n_waves) {
        const uint32_t p0 = n_heavy + task * lc, p1 = min(n_walk, p0 + lc);
        auto place = [&](uint32_t p) { return a.order[min(p, p1 - 1u) + zero]; };
        auto head = [&](uint32_t x, LightHead& h) {
            h.x = x;
            h.a0 = a.off[x];
            h.k = a.kx[x];
        };
        // middles of h in the lanes below its count; the others read its
        // first one and hold an empty slice
        auto lanes = [&](const LightHead& h, Mid& m) {
            const uint32_t i = h.a0 + ((uint32_t)lane < h.k ? (uint32_t)lane : 0u);
            m.e = a.ent[i];
            m.cr = a.cross[i];
            m.ms = a.mstart[i];
        };
        LightHead h[2], h2;
        Mid m;
        Flat f[2];
        Group<GP> gr[2];
        uint32_t x3;
        auto begin = [&](int b) {  // lays out the anchor whose middles are in m, loads its first group
            const int32_t len = (uint32_t)lane < h[b].k ? (int32_t)(m.cr - m.ms) : 0;
            flat_begin(f[b], flat[wave][b].tab, m.ms, len, m.e);
            flat_load<GP>(f[b], mark, flat[wave][b].tab, a.ent, 0, gr[b]);
        };
        head(place(p0), h[0]);
        lanes(h[0], m);
        begin(0);
        head(place(p0 + 1), h[1]);
        lanes(h[1], m);
        head(place(p0 + 2), h2);
        x3 = place(p0 + 3);
        uint32_t p = p0;
        // counts anchor b while the next ones are read ahead; every read is
        // used one step after it went out
        auto step = [&](int b) {
            begin(1 - b);
            const uint32_t x = h[b].x;
            const uint32_t rx = x >= (uint32_t)a.n_u ? x - (uint32_t)a.n_u : x;
            const LightHead own = h[b];
            lanes(h2, m);
            h[b] = h2;
            head(x3, h2);
            x3 = place(p + 4);
            __builtin_amdgcn_sched_barrier(0);
            bool full = false;  // no more middles than a counter holds: none overflows
            const SlotLayout sl = slot_layout((uint32_t)__builtin_amdgcn_readfirstlane((int)rx));
            // slots for twice the wedges: most anchors have few, and clearing
            // the whole table took longer than counting them
            const int lt = max(8, 33 - __clz(f[b].total - 1));
            uint32_t s = hash_group<GP, false>(tab, gr[b], rx, lt, sl, full);
            for (int32_t j0 = GP * kWave; j0 < f[b].total; j0 += GP * kWave) {
                flat_load<GP>(f[b], mark, flat[wave][b].tab, a.ent, j0, gr[b]);
                s += hash_group<GP, false>(tab, gr[b], rx, lt, sl, full);
            }
            if constexpr (FULL) {
                if (__any(s != 0u)) {
                    const uint32_t yb = x < (uint32_t)a.n_u ? (uint32_t)a.n_u : 0u;
                    const uint32_t e = a.ent[own.a0 + ((uint32_t)lane < own.k ? (uint32_t)lane : 0u)];
                    hash_credit<GP>(f[b], mark, flat[wave][b].tab, a.ent, tab, rx, lt, sl, ys[wave], a.pv,
                                    yb + top_rank(e));
                    const unsigned long long w = wave_sum((unsigned long long)s);
                    if (lane == 0) atomicAdd(&a.pv[x], w);
                    for (int i = lane; i < (1 << lt); i += kWave) {
                        const uint32_t v = tab[i];
                        if (v) hash_share(v, rx, (uint32_t)a.n_u - yb, sl, a.pv);
                    }
                    __builtin_amdgcn_wave_barrier();
                }
            }
            clear(1 << lt);
            acc += 2u * s;
            return ++p < p1;
        };
        while (step(0) && step(1)) {
        }
    }
    acc = block_sum<kTopLightWG>(acc, red);
    if (threadIdx.x == 0 && acc) atomicAdd(&my_sums(a.st)->total, acc);
}

// ------------------------------------------------------------------ launch

template <int WG, int BW>
static int top_occ() {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_top_bands<WG, BW, false>, WG, 0) != hipSuccess) return 1;
    return n > 0 ? n : 1;
}

template <int WG, int BW>
static void top_launch(const TopArgs& a, int grid, hipStream_t s) {
    hipLaunchKernelGGL((k_top_bands<WG, BW, false>), dim3(grid), dim3(WG), 0, s, a);
}

struct TopShape {
    int wg, band_words;
    int (*occ)();
    void (*launch)(const TopArgs&, int, hipStream_t);
};
#define BBC_TOP(W, B) {W, B, top_occ<W, B>, top_launch<W, B>}
static const TopShape kTopShapes[] = {BBC_TOP(256, 8192),  BBC_TOP(512, 16384),  BBC_TOP(256, 16384),
                                      BBC_TOP(512, 8192),  BBC_TOP(1024, 32768), BBC_TOP(1024, 16384),
                                      BBC_TOP(128, 4096),  BBC_TOP(128, 8192),   BBC_TOP(256, 4096)};
#undef BBC_TOP

static const TopShape& top_shape(int band_words, int wg) {
    for (const TopShape& t : kTopShapes)
        if (t.band_words == band_words && t.wg == wg) return t;
    return kTopShapes[0];
}

int top_blocks_per_cu(int band_words, int wg) { return top_shape(band_words, wg).occ(); }

template <class K>
static int kernel_occ(K* kernel, int wg) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, wg, 0) != hipSuccess) return 1;
    return n > 0 ? n : 1;
}

int top_light_blocks_per_cu() { return kernel_occ(k_top_light<false>, kTopLightWG); }

// Per-vertex output in id order from the counts in rank order.
__global__ void k_top_credit(const unsigned long long* __restrict__ pv, const int32_t* __restrict__ rank, int64_t n_u,
                             int64_t n, unsigned long long* __restrict__ out) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = pv[(i < n_u ? 0 : n_u) + rank[i]];
}

void launch_top_full(int n_cu, const TopArgs& a, const int32_t* rank, int64_t n, unsigned long long* out,
                     hipStream_t s) {
    constexpr int WG = 512, BW = 16384;
    static const int occ0 = kernel_occ(k_top_hash<1024, 15, 4, 16, true>, 1024),
                     occ1 = kernel_occ(k_top_hash<256, 13, 8, 32, true>, 256),
                     occ2 = kernel_occ(k_top_light<true>, kTopLightWG), occ3 = kernel_occ(k_top_bands<WG, BW, true>, WG);
    hipLaunchKernelGGL((k_top_hash<1024, 15, 4, 16, true>), dim3(n_cu * occ0), dim3(1024), 0, s, a, 0);
    hipLaunchKernelGGL((k_top_hash<256, 13, 8, 32, true>), dim3(n_cu * occ1), dim3(256), 0, s, a, 1);
    hipLaunchKernelGGL(k_top_light<true>, dim3(n_cu * occ2), dim3(kTopLightWG), 0, s, a);
    hipLaunchKernelGGL((k_top_bands<WG, BW, true>), dim3(n_cu * occ3), dim3(WG), 0, s, a);
    const int64_t g = (n + 255) / 256;
    hipLaunchKernelGGL(k_top_credit, dim3((unsigned)(g > 4096 ? 4096 : g)), dim3(256), 0, s, a.pv, rank, (int64_t)a.n_u, n,
                       out);
}

// The tiers' kernels: tables of twice the tier's largest work.
void launch_top(int band_words, int wg, int grid, int light_grid, int n_cu, const TopArgs& a, hipStream_t s) {
    static_assert(kTierWork[0] * 2 == 1u << 15 && kTierWork[1] * 2 == 1u << 13, "table sizes");
    static const int occ0 = kernel_occ(k_top_hash<1024, 15, 4, 16, false>, 1024),
                     occ1 = kernel_occ(k_top_hash<256, 13, 8, 32, false>, 256);
    hipLaunchKernelGGL((k_top_hash<1024, 15, 4, 16, false>), dim3(n_cu * occ0), dim3(1024), 0, s, a, 0);
    hipLaunchKernelGGL((k_top_hash<256, 13, 8, 32, false>), dim3(n_cu * occ1), dim3(256), 0, s, a, 1);
    hipLaunchKernelGGL(k_top_light<false>, dim3(light_grid), dim3(kTopLightWG), 0, s, a);
    top_shape(band_words, wg).launch(a, grid, s);
}

}  // namespace bbc
