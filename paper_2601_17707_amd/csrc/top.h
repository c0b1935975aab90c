// Declarations of the top-vertex pipeline (top_build.hip, top_walk.hip).
//
// Every butterfly u1 - v1 - u2 - v2 is counted once, from its highest vertex
// x in one order of all vertices of both sides (degree class, then side, then
// id): the wedges x - y - w with y and w both below x.  A pair {x, w} with
// a agreeing and b disagreeing such wedges adds C(a,2) + C(b,2) (Lemma 1).
// Restricting the middle as well as the endpoint is the vertex-priority rule
// of the butterfly-counting literature (Wang et al., "Vertex Priority Based
// Butterfly Counting", PVLDB 2019); the signs do not enter the choice.  A hub
// is then never the middle of its own neighbours' wedges: the power-law graph
// of 20M edges walks 3.35e9 wedges instead of the 1.98e10 of one fixed anchor
// side.
//
// Vertices of both sides share one numbering: U ranks [0, n_u), then V ranks
// n_u + [0, n_v), each side ranked by (degree class, id).  Lists of both
// sides share arrays of 2 m entries, U lists first: ent[p] = rank of the
// neighbour on its own side | negative << 31, ascending in rank inside a list;
// cross[p] = where the same edge stands in the neighbour's list.
#pragma once

#include <algorithm>

#include "bbc_internal.h"
#include "route.h"

namespace bbc {

__host__ __device__ __forceinline__ uint32_t top_rank(uint32_t e) { return e & 0x7fffffffu; }

// Degree class: exact below 16, then three bits below the leading one; 232
// classes for any 31-bit degree, so one 8-bit radix pass orders a side.
constexpr uint32_t kDegClasses = 256;
__host__ __device__ __forceinline__ uint32_t degree_class(uint32_t d) {
    if (d < 16u) return d;
    const int e = 31 - __builtin_clz(d);
    return 16u + ((uint32_t)(e - 4) << 3) + ((d >> (e - 3)) & 7u);
}

// Counter bands over the endpoint ranks of one side.  The
// common neighbours of x and w number at most deg(w), so the counter width
// follows the endpoint's degree: ranks of degree <= 15 lie in bands of 4-bit
// pairs, then 8, 16 and 32 bits (modes 0-3).  end: the side's ranks; s1, s2,
// s3: first rank of modes 1, 2, 3; c1, c2, c3: first band of them.
struct TopBands {
    int32_t s1, s2, s3, end;
    int32_t c1, c2, c3, nb;
    int32_t lw;  // log2 of the counter words per band
};

__device__ __forceinline__ int band_mode(const TopBands& B, int32_t b) {
    return b < B.c1 ? 0 : b < B.c2 ? 1 : b < B.c3 ? 2 : 3;
}
__device__ __forceinline__ int32_t band_of(const TopBands& B, int32_t r) {
    if (r < B.s1) return r >> (B.lw + 2);
    if (r < B.s2) return B.c1 + ((r - B.s1) >> (B.lw + 1));
    if (r < B.s3) return B.c2 + ((r - B.s2) >> B.lw);
    return B.c3 + ((r - B.s3) >> (B.lw - 1));
}
// First rank of band b (the side's end for b >= nb).
__device__ __forceinline__ int32_t band_lo(const TopBands& B, int32_t b) {
    if (b >= B.nb) return B.end;
    if (b < B.c1) return b << (B.lw + 2);
    if (b < B.c2) return B.s1 + ((b - B.c1) << (B.lw + 1));
    if (b < B.c3) return B.s2 + ((b - B.c2) << B.lw);
    return B.s3 + ((b - B.c3) << (B.lw - 1));
}

// Slots of the hashed tables: 32 bits, a key (anchor rank minus endpoint rank)
// above two counters.  An anchor of rank below 2^20 leaves each counter 6 bits;
// every four times as many ranks take one bit of each, down to 2 bits below
// 2^28.  With 6 bits only, every anchor beyond 2^20 had to be counted in bands,
// most of them empty, however few its wedges (they are the vertices of highest
// degree): 2.5M x 1.25M vertices and 20M edges took 97.5 ms (uniform) and
// 127 ms (power law) instead of 3.1 and 10.5 ms; the one-sided walk, whose wave
// regime ends at 2^20 ranks too, takes 20 and 71 ms.
constexpr uint32_t kSlotBits = 6, kSlotMinBits = 2;
static_assert(kTopMaxSide == 1ll << (32 - 2 * kSlotMinBits), "the widest side's keys fit a slot");
__host__ __device__ __forceinline__ uint32_t slot_bits(uint32_t rank) {  // per counter
    const uint32_t b = (uint32_t)__builtin_clz(rank | 1u) >> 1;
    return b < kSlotBits ? b : kSlotBits;
}

// Schedule classes (sort key of the anchors): descending work class, then
// the wave regime, then anchors with fewer than two wedges.
constexpr uint32_t kTopLight = 254, kTopNone = 255;

// Work tiers of the workgroup regime: anchors of at least kTierWork[0] wedges
// are counted in bands, those from kTierWork[1] and those below it in hashed
// tables of 32K and 8K slots.
constexpr int kTopTiers = 2;
constexpr uint32_t kTierWork[kTopTiers] = {16384, 4096};

// Positions in the schedule: [0, n_tier[0]) the anchors counted in bands,
// [n_tier[i], n_tier[i + 1]) tier i, [n_tier[kTopTiers], n_walk) the wave
// regime.  n_extra anchors whose hashed counters overflowed join the bands.
struct TopCounts {
    uint32_t n_tier[kTopTiers + 1], n_walk, nb_max, n_extra;
    unsigned long long queue[8];  // an anchor has a task per band: more than 2^32 on the widest sides
    unsigned int queue_hash[kTopTiers];
};

constexpr uint32_t kNoIndex = 0xffffffffu;

// What the walk kernels read.
struct TopArgs {
    const uint32_t *ent, *cross, *mstart, *mbase, *off, *kx, *order, *idx;
    const unsigned long long* work;
    const TopBands* bands;   // [side]
    DevStatus* st;
    TopCounts* tc;
    uint32_t* extra;         // anchors left to the bands by the hashed kernels
    unsigned long long* pv;  // per-vertex counts in rank order (FULL kernels)
    int32_t n_u;
    int32_t statik, queue_chunk, light_chunk;
};

// Device buffers of the build.
struct TopBuild {
    uint32_t *deg, *key, *inv, *vk_a, *vv_a, *degr, *off, *thr, *kx, *order, *ioff, *icnt;
    int32_t* rank;
    uint32_t *first, *last;
    unsigned long long* work;
    uint32_t* cstart;
    TopBands* bands;
    uint32_t *ent, *cross, *mstart, *e, *idx;
    uint2* row;
    unsigned long long* pv;
    TopCounts* tc;
};

void top_vertex_u(const int32_t* off, int32_t n_u, int64_t m, uint32_t* deg, uint32_t* key, DevStatus* st,
                  hipStream_t s);
void top_decode(const int32_t* off, const int32_t* adj, const int8_t* sg, int32_t n_u, int32_t n_v, int64_t m,
                int check_sign, const int32_t* rank, const uint32_t* roff, DevStatus* st, uint32_t* key, uint32_t* pay,
                hipStream_t s);
void top_runs(const uint32_t* key, const uint32_t* pay, int64_t m, int64_t n_v, uint32_t* first, uint32_t* last,
              uint32_t* deg, uint32_t* vkey, DevStatus* st, hipStream_t s);
void top_ranks(const uint32_t* inv, const uint32_t* deg, int64_t n, int side, int32_t* rank, uint32_t* degr,
               uint32_t* cstart, hipStream_t s);
void top_move(const uint32_t* key, const uint32_t* pay, int64_t m, const uint32_t* first, const int32_t* rank,
              const uint32_t* voff, uint32_t* lv, uint32_t* pay2, const DevStatus* st, hipStream_t s);
void top_vertices(const uint32_t* degr, const uint32_t* cstart, int64_t n_u, int64_t n_v, int s_is_u, int lw,
                  uint32_t* thr, uint32_t* kx, unsigned long long* work, TopBands* bands, TopCounts* tc, DevStatus* st,
                  hipStream_t s);
void top_index(const uint32_t* off, int64_t n_u, int64_t n, const TopBands* bands, uint32_t* icnt, uint32_t* ioff,
               uint2* row, uint32_t* partials, const DevStatus* st, hipStream_t s);
void top_work(const uint32_t* xkey, const uint32_t* vpay, const uint32_t* ent, const uint32_t* cross, const uint2* row,
              const uint32_t* thr, const TopBands* bands, int64_t m, int32_t n_u, uint32_t* idx, uint32_t* mstart,
              uint32_t* mbase, uint32_t* kx, unsigned long long* work, const DevStatus* st, hipStream_t s);
void top_schedule(const unsigned long long* work, const uint32_t* kx, int64_t n_u, int64_t n, uint32_t light_w,
                  uint32_t* skey, const DevStatus* st, hipStream_t s);
void top_counts(const uint32_t* sorted, int64_t n, TopCounts* tc, hipStream_t s);
// Per-vertex counts too, into out (id order); rank: of U ids, then of V ids.
void launch_top_full(int n_cu, const TopArgs& a, const int32_t* rank, int64_t n, unsigned long long* out,
                     hipStream_t s);
void launch_top(int band_words, int wg, int grid, int light_grid, int n_cu, const TopArgs& a, hipStream_t s);
int top_blocks_per_cu(int band_words, int wg);
int top_light_blocks_per_cu();

}  // namespace bbc
