// Build of the top-vertex pipeline (top.h): both sides ranked by degree
// class, both sides' lists sorted by rank, cross positions between them, and
// the schedule of the walk.
//
// The edges are decoded straight into U-rank order (rows move as a whole), so
// one stable sort by V id leaves every V list sorted by U rank; its runs give
// the V degrees.  The V lists move to V-rank order and one stable sort by U
// rank, carrying each entry's position, leaves every U list sorted by V rank
// together with both directions of the cross positions.
//
// Every kernel after the input checks first reads the status flags and does
// nothing once an input error is flagged.
#include "top.h"

namespace bbc {

__device__ __forceinline__ void top_flag(DevStatus* st, int32_t bit, int64_t* slot, int64_t idx) {
    atomicOr(&st->flags, bit);
    atomicMin((unsigned long long*)slot, (unsigned long long)idx);
}

__device__ __forceinline__ bool top_bad(const DevStatus* st) { return *(volatile const int32_t*)&st->flags != 0; }

#define TOP_STRIDE(i, n)                                                        \
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n); \
         i += (int64_t)gridDim.x * blockDim.x)

static int top_grid(int64_t n, int threads, int cap = 16384) {
    int64_t g = (n + threads - 1) / threads;
    return (int)(g < 1 ? 1 : g > cap ? cap : g);
}

// Offset checks (offsets[0] == 0, offsets[n_u] == m, non-decreasing), U
// degrees and their sort keys.
__global__ void k_top_vertex_u(const int32_t* __restrict__ off, int32_t n_u, int64_t m, uint32_t* __restrict__ deg,
                               uint32_t* __restrict__ key, DevStatus* st) {
    TOP_STRIDE(i, (int64_t)n_u + 1) {
        const int32_t o = off[i];
        const int32_t nx = i < n_u ? off[i + 1] : o;
        if ((i == 0 && o != 0) || (i == n_u && (int64_t)o != m) || nx < o) top_flag(st, kBadOffsets, &st->bad_offset, i);
        if (i < n_u) {
            const uint32_t d = nx > o ? (uint32_t)(nx - o) : 0u;
            deg[i] = d;
            key[i] = degree_class(d);
        }
    }
}

// Runs of the edges sorted by V id: first and past-the-last position of every
// id; inside a run the U ranks ascend, so a repeated pair is two equal
// neighbours.
__global__ void k_top_runs(const uint32_t* __restrict__ key, const uint32_t* __restrict__ pay, int64_t m,
                           uint32_t* __restrict__ first, uint32_t* __restrict__ last, DevStatus* st) {
    if (top_bad(st)) return;
    TOP_STRIDE(p, m) {
        const uint32_t k = key[p];
        const bool end = p == m - 1 || key[p + 1] != k;
        if (p == 0 || key[p - 1] != k) first[k] = (uint32_t)p;
        if (end) last[k] = (uint32_t)(p + 1);
        else if (top_rank(pay[p]) == top_rank(pay[p + 1])) top_flag(st, kBadDup, &st->bad_dup, p);
    }
}

// V degrees (last is zero for ids that never occur) and their sort keys.
__global__ void k_top_vertex_v(const uint32_t* __restrict__ first, const uint32_t* __restrict__ last, int64_t n_v,
                               uint32_t* __restrict__ deg, uint32_t* __restrict__ key) {
    TOP_STRIDE(v, n_v) {
        const uint32_t e = last[v];
        const uint32_t d = e ? e - first[v] : 0u;
        deg[v] = d;
        key[v] = degree_class(d);
    }
}

// Ranks of one side from its ids in (class, id) order, degrees by rank, and
// the first rank of every degree class: cstart[side * 257 + class], with entry
// 256 the end.
__global__ void k_top_ranks(const uint32_t* __restrict__ inv, const uint32_t* __restrict__ deg, int64_t n, int side,
                            int32_t* __restrict__ rank, uint32_t* __restrict__ degr, uint32_t* __restrict__ cstart) {
    uint32_t* cs = cstart + side * (int)(kDegClasses + 1);
    TOP_STRIDE(r, n) {
        const uint32_t id = inv[r];
        const uint32_t d = deg[id];
        rank[id] = (int32_t)r;
        degr[r] = d;
        const int c = (int)degree_class(d);
        const int cp = r > 0 ? (int)degree_class(deg[inv[r - 1]]) : -1;
        for (int k = cp + 1; k <= c; ++k) cs[k] = (uint32_t)r;
        if (r == n - 1)
            for (int k = c + 1; k <= (int)kDegClasses; ++k) cs[k] = (uint32_t)n;
    }
}

// V lists in rank order: the run of each V id moves, in its order, to its
// rank's place.  pay2 is the payload of the sort by U rank: V rank | neg << 31.
__global__ void k_top_move(const uint32_t* __restrict__ key, const uint32_t* __restrict__ pay, int64_t m,
                           const uint32_t* __restrict__ first, const int32_t* __restrict__ rank,
                           const uint32_t* __restrict__ voff, uint32_t* __restrict__ lv, uint32_t* __restrict__ pay2,
                           const DevStatus* st) {
    if (top_bad(st)) return;
    constexpr int U = 4;  // entries per thread whose gathers are in flight together
    const int64_t stride = (int64_t)gridDim.x * blockDim.x * U;
    for (int64_t p0 = (int64_t)blockIdx.x * blockDim.x * U + threadIdx.x; p0 < m; p0 += stride) {
        uint32_t v[U], c[U], f[U], o[U], r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t p = p0 + (int64_t)u * blockDim.x;
            v[u] = p < m ? key[p] : 0u;
            c[u] = p < m ? pay[p] : 0u;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            r[u] = (uint32_t)rank[v[u]];
            f[u] = first[v[u]];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) o[u] = p0 + (int64_t)u * blockDim.x < m ? voff[r[u]] : 0u;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t p = p0 + (int64_t)u * blockDim.x;
            if (p < m) {
                const uint32_t q = o[u] - (uint32_t)m + ((uint32_t)p - f[u]);  // voff counts from m
                lv[q] = c[u];
                pay2[q] = r[u] | (c[u] & 0x80000000u);
            }
        }
    }
}

// Per vertex x: thr[x] = first rank of the other side that is not below x (a
// vertex is below x if its degree class is lower; at equal classes U is below
// V), so its middles are the entries of its list below thr[x].  Also clears
// what later kernels accumulate, lays out the counter bands of both sides and
// sums C(deg, 2) over the centre side (the wedges of the statistics).
__global__ __launch_bounds__(256) void k_top_vertices(const uint32_t* __restrict__ degr,
                                                      const uint32_t* __restrict__ cstart, int64_t n_u, int64_t n_v,
                                                      int s_is_u, int lw, uint32_t* __restrict__ thr,
                                                      uint32_t* __restrict__ kx,
                                                      unsigned long long* __restrict__ work,
                                                      TopBands* __restrict__ bands, TopCounts* tc, DevStatus* st) {
    __shared__ unsigned long long red[256 / kWave];
    const int64_t n = n_u + n_v;
    unsigned long long wedges = 0;
    const bool bad = top_bad(st);
    if (!bad) {
        TOP_STRIDE(x, n) {
            const int side = x >= n_u;
            const uint32_t d = degr[x];
            thr[x] = cstart[(1 - side) * (int)(kDegClasses + 1) + degree_class(d) + side];
            kx[x] = 0;
            work[x] = 0;
            if (side == s_is_u) wedges += (unsigned long long)d * (d - (d > 0)) / 2ull;
        }
    }
    wedges = block_sum<256>(wedges, red);
    if (threadIdx.x == 0 && wedges) {
        atomicAdd(&my_sums(st)->wedges, wedges);
        atomicAdd(&my_sums(st)->walked, wedges);
    }
    if (blockIdx.x == 0 && threadIdx.x < 2) {
        const int side = threadIdx.x;
        TopBands B;
        B.lw = lw;
        B.end = (int32_t)(side ? n_v : n_u);
        B.s1 = B.s2 = B.s3 = B.end;
        B.c1 = B.c2 = B.c3 = B.nb = 0;
        if (!bad) {
            const uint32_t* cs = cstart + side * (int)(kDegClasses + 1);
            const int64_t lim[3] = {cs[degree_class(16)], cs[degree_class(256)], cs[degree_class(65536)]};
            int64_t at = 0, nb = 0;
            int64_t s[4], c[4];
            for (int k = 0; k < 4; ++k) {
                s[k] = at;
                c[k] = nb;
                const int sh = lw + 2 - k;  // log2 of the ranks per band
                const int64_t top = k < 3 ? lim[k] : B.end;
                // whole bands below the section's limit (all ranks when it reaches the end)
                const int64_t cnt = top >= B.end ? (B.end - at + (1ll << sh) - 1) >> sh : (top - at) >> sh;
                nb += cnt;
                at = at + (cnt << sh) < B.end ? at + (cnt << sh) : B.end;
            }
            B.s1 = (int32_t)s[1];
            B.s2 = (int32_t)s[2];
            B.s3 = (int32_t)s[3];
            B.c1 = (int32_t)c[1];
            B.c2 = (int32_t)c[2];
            B.c3 = (int32_t)c[3];
            B.nb = (int32_t)nb;
            atomicMax(&tc->nb_max, (uint32_t)nb);
        }
        bands[side] = B;
    }
}

// ------------------------------------------------------------- band index
//
// A list of side A is walked in bands of B ranks: idx[ioff[y] + b] = first
// position of list y with a rank in band b or above, b = 0 .. nb.  Where there
// are more than kTopFewBands bands only lists with at least nb entries are
// indexed (the walk searches the shorter ones); index_words bounds the entries.

__global__ void k_top_idx_count(const uint32_t* __restrict__ off, int64_t n_u, int64_t n,
                                const TopBands* __restrict__ bands, uint32_t* __restrict__ cnt, const DevStatus* st) {
    const bool bad = top_bad(st);
    TOP_STRIDE(y, n) {
        uint32_t c = 0;
        if (!bad) {
            const uint32_t len = off[y + 1] - off[y], nb = (uint32_t)bands[y < n_u ? 1 : 0].nb;
            if (nb > 1 && (len >= nb || (len > 0 && nb <= (uint32_t)kTopFewBands))) c = nb + 1;
        }
        cnt[y] = c;
    }
}

// List of entry p: the sort key of the U lists (rank | neg << 31), the second
// sort's payload for the V lists.
__device__ __forceinline__ uint32_t list_of(const uint32_t* xkey, const uint32_t* vpay, int64_t m, uint32_t n_u,
                                            int64_t p) {
    return p < m ? top_rank(xkey[p]) : n_u + top_rank(vpay[p - m]);
}

// What a list's users need of it, in one 8-byte word: its start and its index
// row (kNoIndex without one).
__global__ void k_top_rows(const uint32_t* __restrict__ off, const uint32_t* __restrict__ ioff, int64_t n,
                           uint2* __restrict__ row, const DevStatus* st) {
    if (top_bad(st)) return;
    TOP_STRIDE(y, n) row[y] = uint2{off[y], ioff[y + 1] != ioff[y] ? ioff[y] : kNoIndex};
}

// ------------------------------------------------------------------- work

// Per list entry p of vertex x: the index entries of x's list between the
// bands of entry p - 1 and entry p; and if p is a middle of x: mstart[p] =
// start of the middle's list, mbase[p] = its index row, and its wedges,
// cross[p] - mstart[p], added to work[x]; kx[x] = number of middles.  Whole
// waves take 64 consecutive entries: neighbours from the lanes beside, prefix
// sums over the lanes and one atomic per vertex and wave.  Bound by the random
// read per middle (20M power-law edges: one 8-byte row instead of three words
// from two arrays, and the index filled on the way instead of by a kernel of
// its own that read the entries again: 619 us instead of 558 + 270 us).  Many
// workgroups of two entries a thread hide its latency better than 2048 of four
// in a loop: 492 and 627 us there, 437 and 609 us on 20M uniform edges.
constexpr int kTopWorkItems = 2;  // entries per thread whose loads are in flight together
__global__ __launch_bounds__(256) void k_top_work(const uint32_t* __restrict__ xkey, const uint32_t* __restrict__ vpay,
                                                  const uint32_t* __restrict__ ent, const uint32_t* __restrict__ cross,
                                                  const uint2* __restrict__ row, const uint32_t* __restrict__ thr,
                                                  const TopBands* __restrict__ bands, int64_t m, int32_t n_u,
                                                  uint32_t* __restrict__ idx, uint32_t* __restrict__ mstart,
                                                  uint32_t* __restrict__ mbase, uint32_t* __restrict__ kx,
                                                  unsigned long long* __restrict__ work, const DevStatus* st) {
    if (top_bad(st)) return;
    constexpr int U = kTopWorkItems;
    constexpr uint32_t kNone = 0xffffffffu;
    const int lane = lane_id();
    const TopBands BU = bands[0], BV = bands[1];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x * U;
    for (int64_t p0 = (int64_t)blockIdx.x * blockDim.x * U; p0 < 2 * m; p0 += stride) {
        uint32_t x[U], e[U], cr[U], xs[U], es[U];
        bool mid[U];
        uint2 r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t p = p0 + u * blockDim.x + threadIdx.x;
            x[u] = xs[u] = kNone;
            e[u] = cr[u] = es[u] = 0;
            if (p < 2 * m) {
                x[u] = list_of(xkey, vpay, m, (uint32_t)n_u, p);
                e[u] = ent[p];
                cr[u] = cross[p];
            }
            // the entries beside the wave's: before its first lane, after its last
            const int64_t q = lane == 0 ? p - 1 : p + 1;
            if ((lane == 0 || lane == kWave - 1) && q >= 0 && q < 2 * m) {
                xs[u] = list_of(xkey, vpay, m, (uint32_t)n_u, q);
                es[u] = ent[q];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) mid[u] = x[u] != kNone && top_rank(e[u]) < thr[x[u]];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            r[u] = uint2{0u, 0u};
            if (mid[u]) r[u] = row[(x[u] < (uint32_t)n_u ? (uint32_t)n_u : 0u) + top_rank(e[u])];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t p = p0 + u * blockDim.x + threadIdx.x;
            const uint32_t w = mid[u] ? cr[u] - r[u].x : 0u;
            if (mid[u]) {
                mstart[p] = r[u].x;
                mbase[p] = r[u].y;
            }
            const bool lu = x[u] < (uint32_t)n_u;
            const TopBands& B = lu ? BV : BU;
            uint32_t xp = (uint32_t)__shfl_up((int)x[u], 1, kWave), xn = (uint32_t)__shfl_down((int)x[u], 1, kWave);
            uint32_t ep = (uint32_t)__shfl_up((int)e[u], 1, kWave);
            int mn = __shfl_down((int)mid[u], 1, kWave);
            if (lane == 0) {
                xp = xs[u];
                ep = es[u];
            }
            if (lane == kWave - 1) {
                xn = xs[u];
                mn = mid[u] && xn == x[u] && top_rank(es[u]) < thr[x[u]];
            }
            if (x[u] != kNone && B.nb > 1) {
                const bool start = xp != x[u], end = xn != x[u];
                const int32_t b = band_of(B, (int32_t)top_rank(e[u]));
                const int32_t bp = start ? -1 : band_of(B, (int32_t)top_rank(ep));
                if (b != bp || end) {
                    const uint32_t i0 = row[x[u]].y;
                    if (i0 != kNoIndex) {
                        for (int32_t k = bp + 1; k <= b; ++k) idx[i0 + k] = (uint32_t)p;
                        if (end)
                            for (int32_t k = b + 1; k <= B.nb; ++k) idx[i0 + k] = (uint32_t)(p + 1);
                    }
                }
            }
            if (mid[u] && (xn != x[u] || !mn)) kx[x[u]] = (uint32_t)(p + 1) - row[x[u]].x;
            // inclusive sums over the lanes in two halves of 16 bits, then
            // the difference over each run of one vertex at its last lane
            const uint32_t lo = wave_inclusive_sum_dpp(w & 0xffffu), hi = wave_inclusive_sum_dpp(w >> 16);
            const unsigned long long heads = __ballot(lane == 0 || xp != x[u]);
            const int h = 63 - __clzll(heads & (~0ull >> (63 - lane)));
            const uint32_t plo = (uint32_t)__shfl((int)lo, h > 0 ? h - 1 : 0, kWave);
            const uint32_t phi = (uint32_t)__shfl((int)hi, h > 0 ? h - 1 : 0, kWave);
            const unsigned long long run = ((unsigned long long)(hi - (h > 0 ? phi : 0u)) << 16) + (lo - (h > 0 ? plo : 0u));
            const bool last = lane == kWave - 1 || ((heads >> (lane + 1)) & 1ull);
            if (x[u] != kNone && last && run) atomicAdd(&work[x[u]], run);
        }
    }
}

// Schedule key of each vertex (see kTopLight): anchors of the workgroup
// regime by descending work class, then the wave regime (at most light_w
// wedges, and as many middles as a slot's counter holds, so that none can
// overflow: 63 below rank 2^20), then anchors without a pair.
__global__ void k_top_schedule(const unsigned long long* __restrict__ work, const uint32_t* __restrict__ kx,
                               int64_t n_u, int64_t n, uint32_t light_w, uint32_t* __restrict__ skey,
                               const DevStatus* st) {
    const bool bad = top_bad(st);
    TOP_STRIDE(x, n) {
        uint32_t key = kTopNone;
        if (!bad) {
            const unsigned long long w = work[x];
            const uint32_t k = kx[x];
            if (w >= 2 && k >= 2) {
                const uint32_t most = (1u << slot_bits((uint32_t)(x >= n_u ? x - n_u : x))) - 1u;
                const uint32_t c = degree_class(w > 0x7fffffffull ? 0x7fffffffu : (uint32_t)w);
                key = w <= light_w && k <= most ? kTopLight : 231u - c;
            }
        }
        skey[x] = key;
    }
}

// Boundaries of the schedule from its sorted keys.
__global__ __launch_bounds__(256) void k_top_counts(const uint32_t* __restrict__ sorted, int64_t n, TopCounts* tc) {
    TOP_STRIDE(i, n) {
        const uint32_t k = sorted[i], kn = i + 1 < n ? sorted[i + 1] : 256u;
        if (k == kn) continue;
#pragma unroll
        for (int t = 0; t < kTopTiers; ++t) {
            const uint32_t cut = 231u - degree_class(kTierWork[t]);
            if (k <= cut && kn > cut) tc->n_tier[t] = (uint32_t)(i + 1);
        }
        if (k <= 231u && kn > 231u) tc->n_tier[kTopTiers] = (uint32_t)(i + 1);
        if (k <= kTopLight && kn > kTopLight) tc->n_walk = (uint32_t)(i + 1);
    }
}

// ------------------------------------------------------------ host launchers

void top_vertex_u(const int32_t* off, int32_t n_u, int64_t m, uint32_t* deg, uint32_t* key, DevStatus* st,
                  hipStream_t s) {
    hipLaunchKernelGGL(k_top_vertex_u, dim3(top_grid((int64_t)n_u + 1, 256)), dim3(256), 0, s, off, n_u, m, deg, key,
                       st);
}

void top_runs(const uint32_t* key, const uint32_t* pay, int64_t m, int64_t n_v, uint32_t* first, uint32_t* last,
              uint32_t* deg, uint32_t* vkey, DevStatus* st, hipStream_t s) {
    fill_u32(last, 0u, n_v, s);
    hipLaunchKernelGGL(k_top_runs, dim3(top_grid(m, 256)), dim3(256), 0, s, key, pay, m, first, last, st);
    hipLaunchKernelGGL(k_top_vertex_v, dim3(top_grid(n_v, 256)), dim3(256), 0, s, first, last, n_v, deg, vkey);
}

void top_ranks(const uint32_t* inv, const uint32_t* deg, int64_t n, int side, int32_t* rank, uint32_t* degr,
               uint32_t* cstart, hipStream_t s) {
    hipLaunchKernelGGL(k_top_ranks, dim3(top_grid(n, 256)), dim3(256), 0, s, inv, deg, n, side, rank, degr, cstart);
}

void top_move(const uint32_t* key, const uint32_t* pay, int64_t m, const uint32_t* first, const int32_t* rank,
              const uint32_t* voff, uint32_t* lv, uint32_t* pay2, const DevStatus* st, hipStream_t s) {
    hipLaunchKernelGGL(k_top_move, dim3(top_grid((m + 3) / 4, 256)), dim3(256), 0, s, key, pay, m, first, rank, voff,
                       lv, pay2, st);
}

void top_vertices(const uint32_t* degr, const uint32_t* cstart, int64_t n_u, int64_t n_v, int s_is_u, int lw,
                  uint32_t* thr, uint32_t* kx, unsigned long long* work, TopBands* bands, TopCounts* tc, DevStatus* st,
                  hipStream_t s) {
    hipLaunchKernelGGL(k_top_vertices, dim3(top_grid(n_u + n_v, 256, 512)), dim3(256), 0, s, degr, cstart, n_u, n_v,
                       s_is_u, lw, thr, kx, work, bands, tc, st);
}

void top_index(const uint32_t* off, int64_t n_u, int64_t n, const TopBands* bands, uint32_t* icnt, uint32_t* ioff,
               uint2* row, uint32_t* partials, const DevStatus* st, hipStream_t s) {
    hipLaunchKernelGGL(k_top_idx_count, dim3(top_grid(n, 256)), dim3(256), 0, s, off, n_u, n, bands, icnt, st);
    scan_exclusive_u32(icnt, ioff, n, partials, s);
    hipLaunchKernelGGL(k_top_rows, dim3(top_grid(n, 256)), dim3(256), 0, s, off, ioff, n, row, st);
}

void top_work(const uint32_t* xkey, const uint32_t* vpay, const uint32_t* ent, const uint32_t* cross, const uint2* row,
              const uint32_t* thr, const TopBands* bands, int64_t m, int32_t n_u, uint32_t* idx, uint32_t* mstart,
              uint32_t* mbase, uint32_t* kx, unsigned long long* work, const DevStatus* st, hipStream_t s) {
    hipLaunchKernelGGL(k_top_work, dim3(top_grid(2 * m, 256 * kTopWorkItems)), dim3(256), 0, s, xkey, vpay, ent, cross, row, thr,
                       bands, m, n_u, idx, mstart, mbase, kx, work, st);
}

void top_schedule(const unsigned long long* work, const uint32_t* kx, int64_t n_u, int64_t n, uint32_t light_w,
                  uint32_t* skey, const DevStatus* st, hipStream_t s) {
    hipLaunchKernelGGL(k_top_schedule, dim3(top_grid(n, 256)), dim3(256), 0, s, work, kx, n_u, n, light_w, skey, st);
}

void top_counts(const uint32_t* sorted, int64_t n, TopCounts* tc, hipStream_t s) {
    hipLaunchKernelGGL(k_top_counts, dim3(top_grid(n, 256, 1024)), dim3(256), 0, s, sorted, n, tc);
}

}  // namespace bbc
