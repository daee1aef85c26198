// Device-side building blocks of one BVC-PLL batch (Algorithm 4), shared by
// the whole-grid kernels of a single large graph (pll_build.hip) and by the
// persistent kernel that builds many graphs, one workgroup per graph
// (pll_multi.hip).  A phase is run by an execution group described by Exec:
// wave w of nw waves; queue counters live in nq shards at qs (32 global
// shards for the whole-grid kernels, one LDS shard for a workgroup), and
// this wave appends to shard `my`, whose queue segments start at
// my * seg.
#pragma once

#include "pll_internal.h"
#include "pll_stats.h"

namespace pll {

// Rows longer than kHeavy are not pushed by the wave that owns them but
// queued as work items of kHeavyItem edges, spread over every wave.
constexpr uint32_t kHeavy = 1024;
constexpr uint32_t kHeavyItem = 256;

struct Exec {
    uint32_t w, nw;   // this wave's index in the group, waves in the group
    Shard* qs;        // queue / statistics shards
    uint32_t nq;      // number of shards
    uint32_t my;      // shard this wave appends to
    uint32_t seg;     // entries per shard segment of recv / touched / tstart
    uint32_t zero_i;  // shard this thread clears when a phase resets counters (>= nq: none)
    uint32_t arena_sh;  // first arena region to try
};

// Add the wave's counts since the last call to the workgroup's 64-bit totals
// `tot` (LDS).  The whole wave calls it.
__device__ inline void fold_counts(PhaseStats& st, unsigned long long* tot) {
    unsigned long long v[kCounts];
    take_counts(st, v);
    const uint32_t lane = lane_id();
#pragma unroll
    for (int k = 0; k < kCounts; ++k) {
        if (!ballot64(v[k] != 0)) continue;
        const unsigned long long t = wave_sum64_dpp(v[k]);
        if (lane == 0) atomicAdd(&tot[k], t);
    }
}

// Bit 7 of each byte of the result: that byte of x is <= t, where
// tt = t * 0x01010101 (t <= 254).  Bytes are compared without carries
// between them: s holds, in bit 7 of each byte, [low 7 bits of t >= low 7
// bits of x]; the high bits decide the rest.
__device__ inline uint32_t le4_flags(uint32_t x, uint32_t tt) {
    const uint32_t H = 0x80808080u;
    const uint32_t s = (tt | H) - (x & ~H);
    return ((tt & ~x) | (~(tt ^ x) & s)) & H;
}

// The flags of two words (bits 7, 15, 23, 31 of a and of b) as 8 bits, a's
// in bits 0..3: one multiply gathers both, since with a's flags moved to
// bits 0, 8, 16, 24 and b's to 4, 12, 20, 28, every cross term of the
// product lands below bit 24 or above bit 31, each on a bit of its own.
__device__ inline uint32_t gather8(uint32_t a, uint32_t b) {
    return (((a >> 7) | (b >> 3)) * 0x01020408u) >> 24;
}

// The 16 flags of a 16-byte quarter, byte i in bit i.
__device__ inline uint32_t gather16(uint32_t fx, uint32_t fy, uint32_t fz, uint32_t fw) {
    return gather8(fx, fy) | (gather8(fz, fw) << 8);
}

// Bit i of the result: table byte p[i] <= t, for 64 consecutive bytes.
__device__ inline uint64_t le_mask64(const uint8_t* p, uint32_t tt) {
    const uint4* q = reinterpret_cast<const uint4*>(p);
    uint64_t m = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint4 v = q[i];
        const uint32_t b = gather16(le4_flags(v.x, tt), le4_flags(v.y, tt), le4_flags(v.z, tt), le4_flags(v.w, tt));
        m |= (uint64_t)b << (16 * i);
    }
    return m;
}

// le_mask64 for thresholds t <= kSmallT, with tt1 = (t + 1) * 0x01010101:
// every byte of x | 0x80 is at least 128 > t + 1, so the subtraction
// borrows within no byte, and bit 7 of the difference is clear exactly when
// the byte's low 7 bits are <= t; a byte with bit 7 set (128..255) is above
// t.  Four instructions per word instead of le4_flags's seven.
constexpr uint32_t kSmallT = 126;

// bit 7 of each byte of the result: that byte of x is <= t
__device__ inline uint32_t le4s_flags(uint32_t x, uint32_t tt1) {
    const uint32_t H = 0x80808080u;
    return ~(((x | H) - tt1) | x) & H;
}

__device__ inline uint64_t le_mask64s(const uint8_t* p, uint32_t tt1) {
    const uint4* q = reinterpret_cast<const uint4*>(p);
    uint32_t half[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint4 v0 = q[2 * h], v1 = q[2 * h + 1];
        const uint32_t b0 = gather16(le4s_flags(v0.x, tt1), le4s_flags(v0.y, tt1), le4s_flags(v0.z, tt1),
                                     le4s_flags(v0.w, tt1));
        const uint32_t b1 = gather16(le4s_flags(v1.x, tt1), le4s_flags(v1.y, tt1), le4s_flags(v1.z, tt1),
                                     le4s_flags(v1.w, tt1));
        half[h] = b0 | (b1 << 16);
    }
    return ((uint64_t)half[1] << 32) | half[0];
}

// The segment compare of the scans: SMALLT (every threshold <= kSmallT) takes
// le_mask64s with tt = (t + 1) * 0x01010101, else le_mask64 with t * 0x01010101.
template <bool SMALLT>
__device__ inline uint32_t seg_tt(uint32_t t) {
    return (SMALLT ? t + 1u : t) * 0x01010101u;
}

template <bool SMALLT>
__device__ inline uint64_t seg_le(const uint8_t* p, uint32_t tt) {
    return SMALLT ? le_mask64s(p, tt) : le_mask64(p, tt);
}

// OR over the 64 lanes (DPP wave reduction, the whole wave active); the
// result is wave-uniform.
__device__ inline uint64_t wave_or64_u(uint64_t x) {
    const uint32_t lo = wave_or32_dpp((uint32_t)x);
    const uint32_t hi = wave_or32_dpp((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Scan the label list arena[off .. off+len) of one vertex v.  Lane w (< W)
// holds candidate word cw = bits k of batch vertices u_{64w+k} that arrived
// at distance j.  Returns, in lane w, the candidates of word w for which some
// entry (h, d) of the list with d < j has T[h][k] + d <= j, i.e. the distance
// j is already covered through a hub ranked above u_k (the pruning test of
// Algorithm 4).
// With `relaxed`, entries whose hub is in the current batch are skipped.
// Each chunk of 64 entries makes one pass per candidate word that still
// holds live candidates, and the wave OR-reduces that word's prunes in the
// pass, so the scan stops after the first chunk that leaves no candidate
// live (the top-ranked hubs of the first chunk prune most candidates of the
// late rounds).  The next chunk's entries are loaded while this chunk's
// segments are.  A segment is loaded whole when any of its 16-byte quarters
// holds an entry (row mask): fewer, wider loads than with a gate per quarter.
template <int WM, bool SMALLT = false>
__device__ inline uint64_t prune_scan(const BuildArgs& A, uint64_t off, uint32_t len, uint32_t j, uint64_t cw,
                                      bool relaxed, uint32_t ib, PhaseStats& st) {
    const uint32_t lane = lane_id();
    uint64_t pw = 0;
    // the next chunk's entry is loaded while this chunk's table segments are
    uint32_t next = lane < len ? A.arena[off + lane] : 0u;
    for (uint32_t base = 0; base < len; base += 64) {
        const uint32_t idx = base + lane;
        bool ok = idx < len;
        st.read += ok;
        const uint32_t ent = next;
        next = idx + 64 < len ? A.arena[off + idx + 64] : 0u;
        const uint32_t h = ent >> 8, d = ent & 255u;
        ok = ok && d < j;
        if (relaxed) ok = ok && h < ib;
        const uint64_t rm = ok ? A.rmchk[h] : 0ull;
        // threshold at most 254, the largest finite table byte: at round 255
        // (which only reports the overflow) an empty cell must not prune
        const uint32_t tt = ok ? seg_tt<SMALLT>(min(j - d, PLL_INF8 - 1u)) : 0u;
        const uint8_t* row = A.Tchk + (size_t)h * A.bstride;
        // One pass per word that still holds live candidates (a scalar loop
        // over their mask): every lane compares its entry's table segment,
        // and the wave OR-reduces the word's prunes at once.  So the
        // candidates pruned by this chunk (the top-ranked hubs of the first
        // chunk prune most) load no later segments, one copy of the compare
        // serves every word, and no per-word accumulators are kept.
        const uint64_t live_lane = cw & ~pw;
        uint64_t lw = ballot64(live_lane != 0) & (WM >= 64 ? ~0ull : ((1ull << WM) - 1ull));
        while (lw) {
            const uint32_t w = (uint32_t)__builtin_ctzll(lw);
            lw &= lw - 1;
            uint64_t m = 0;
            if ((rm >> (4 * w)) & 15u) {
                m = seg_le<SMALLT>(row + 64u * w, tt);
                st.table += 4;
            }
            // lane w masks the reduced prunes with its live candidates
            const uint64_t red = wave_or64_u(m);
            if (lane == w) pw |= red & live_lane;
        }
        if (!ballot64((cw & ~pw) != 0)) break;
    }
    return pw;
}

// The round-2 check of receiver v through its neighbours.  At distance 2
// only entries (h, 1) of L(v) can prune (the self entry cannot, as in round
// 1), and in an undirected unweighted graph those are exactly the
// neighbours h of v ranked above both v and the end of the current batch
// (lim): the edge is the only shortest h-v path, so h is its top-ranked
// vertex, and h's batch has run (or, inside the current batch, round 1
// accepted (h, 1) unconditionally).  So the rank-space CSR row of v can
// stand in for L(v): the caller takes it when it is the shorter of the two
// (a low-ranked vertex has a few dozen neighbours and hundreds of label
// entries).  Candidate u_k is pruned when T[h][k] <= 1; the table loads,
// which are the same as those of the label scan, and the lane reductions
// are those of prune_scan.
template <int WM, bool SMALLT = false>
__device__ inline uint64_t prune_scan_nbrs(const BuildArgs& A, uint32_t v, uint32_t lim, uint64_t cw,
                                           PhaseStats& st) {
    const uint32_t lane = lane_id();
    uint64_t pw = 0;
    const uint64_t beg = A.rrow[v], end = A.rrow[v + 1];
    const uint32_t tt = seg_tt<SMALLT>(1u);  // T[h][k] <= 2 - 1
    for (uint64_t base = beg; base < end; base += 64) {
        const uint64_t idx = base + lane;
        const uint32_t h = idx < end ? A.rcol[idx] : ~0u;
        const bool ok = h < lim;
        st.read += idx < end;
        const uint64_t rm = ok ? A.rmchk[h] : 0ull;
        const uint8_t* row = A.Tchk + (size_t)(ok ? h : 0u) * A.bstride;
        // one pass per word with live candidates, as in prune_scan
        const uint64_t live_lane = cw & ~pw;
        uint64_t lw = ballot64(live_lane != 0) & (WM >= 64 ? ~0ull : ((1ull << WM) - 1ull));
        while (lw) {
            const uint32_t w = (uint32_t)__builtin_ctzll(lw);
            lw &= lw - 1;
            uint64_t m = 0;
            if ((rm >> (4 * w)) & 15u) {
                m = seg_le<SMALLT>(row + 64u * w, tt);
                st.table += 4;
            }
            // lane w masks the reduced prunes with its live candidates
            const uint64_t red = wave_or64_u(m);
            if (lane == w) pw |= red & live_lane;
        }
        if (!ballot64((cw & ~pw) != 0)) break;
    }
    return pw;
}

// Room for `need` more entries in the list of rank v (capacity doubling;
// cap is its capacity).
// New blocks come from the bump region X.arena_sh of the arena, or from the
// next region with room.  Wave-uniform; returns the list's offset, or ~0
// when every region is exhausted.
__device__ inline uint64_t wave_reserve(const BuildArgs& A, const Exec& X, uint32_t v, uint64_t off, uint32_t len,
                                        uint32_t cap, uint32_t need) {
    if (len + need <= cap) return off;
    uint32_t newcap = max(cap * 2u, (len + need + 15u) & ~15u);
    newcap = max(newcap, 16u);
    unsigned long long nb = ~0ull;
    if (lane_id() == 0) {
        for (uint32_t t = 0; t < PLL_SHARDS; ++t) {
            const uint32_t sh = (X.arena_sh + t) % PLL_SHARDS;
            unsigned long long* top = &A.ctr->sh[sh].arena_top;
            if (__hip_atomic_load(top, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + newcap > A.region_cap) continue;
            const unsigned long long at = atomicAdd(top, (unsigned long long)newcap);
            if (at + newcap <= A.region_cap) {
                nb = A.region_base + (unsigned long long)sh * A.region_cap + at;
                break;
            }
        }
        atomicAdd(&A.ctr->sh[X.arena_sh % PLL_SHARDS].stat[PLL_ST_GROW], 1ull);
    }
    nb = readlane64(nb, 0);
    if (nb == ~0ull) {
        if (lane_id() == 0) atomicOr(&A.ctr->error, PLL_ERR_ARENA);
        return ~0ull;
    }
    for (uint32_t k = lane_id(); k < len; k += 64) A.arena[nb + k] = A.arena[off + k];
    if (lane_id() == 0) {
        A.loff[v] = nb;
        A.lcap[v] = newcap;
    }
    return nb;
}

// Sharded queue enumeration: lane s (< nq) holds the count of shard s;
// `pre` receives its exclusive prefix and the return value the total.
__device__ inline uint32_t shard_prefix(uint32_t cnt_lane, uint32_t& pre) {
    pre = wave_excl_scan32(cnt_lane);
    return readlane32(pre + cnt_lane, 63);
}

// Shard holding global queue position i (wave-uniform i < total).
__device__ inline uint32_t shard_of(uint32_t nq, uint32_t pre_lane, uint32_t i) {
    const uint64_t m = ballot64(lane_id() < nq && pre_lane <= i);
    return 63u - (uint32_t)__builtin_clzll(m);
}

// Wave-aggregated append of the lanes with `take` to a queue counter;
// returns each taking lane's position (seg_base + index).
__device__ inline uint32_t shard_append(uint32_t* counter, bool take, uint64_t seg_base) {
    const uint64_t bal = ballot64(take);
    if (!bal) return 0;
    const uint32_t lane = lane_id();
    const uint32_t leader = (uint32_t)__builtin_ctzll(bal);
    uint32_t base = 0;
    if (lane == leader) base = atomicAdd(counter, (uint32_t)__builtin_popcountll(bal));
    base = readlane32(base, leader);
    return (uint32_t)(seg_base + base + __builtin_popcountll(bal & lanemask_lt()));
}

// Queue the row of active slot `slot` (list q) as kHeavyItem-edge items
// when it is longer than kHeavy.
__device__ inline void enqueue_heavy(const BuildArgs& A, const Exec& X, uint32_t q, uint32_t slot, uint64_t deg) {
    if (deg <= kHeavy) return;
    const uint32_t nch = (uint32_t)((deg + kHeavyItem - 1) / kHeavyItem);
    uint32_t base = 0;
    if (lane_id() == 0) base = atomicAdd(&X.qs[X.my].hq[q], nch);
    base = readlane32(base, 0);
    for (uint32_t c = lane_id(); c < nch; c += 64) A.hq[q][X.my * A.hq_seg + base + c] = make_uint2(slot, c);
}

__device__ inline uint64_t rank_mask(uint32_t rel, uint32_t w) {
    const uint32_t lo = w * 64u;
    if (rel >= lo + 64u) return ~0ull;
    if (rel <= lo) return 0ull;
    return (1ull << (rel - lo)) - 1ull;
}

// Record d(u_k, h) = d (d >= 1) in the bit planes: plane 2 also holds the
// distances of plane 1, so the thresholds 1 and 2 of rounds 2 and 3, which
// carry nearly every check of a small-diameter graph, are one plane each;
// the rare larger thresholds OR the exact planes 3..t on top.  Making planes
// 3 and up cumulative too would cost a second atomic for nearly every entry
// (90% of the R-MAT-20 label entries are at distance 2).
__device__ inline void plane_set(const BuildArgs& A, uint32_t h, uint32_t d, uint32_t k) {
    if (d > PLL_PLANES) return;
    unsigned long long* row =
        reinterpret_cast<unsigned long long*>(A.P) + (size_t)h * (PLL_PLANES * A.W) + (k >> 6);
    const unsigned long long bit = 1ull << (k & 63u);
    if (d == 1) atomicOr(row, bit);
    atomicOr(row + (max(d, 2u) - 1u) * A.W, bit);
}

// Batch initialisation of Algorithm 4: delta L(u) = {(u,0)}, L(u) gets
// (u,0), L(u) -> H(u).
// The initial active list holds batch vertex u_k in slot k.
//
// With planes and HOT, a workgroup runs the kInitRoots consecutive roots of one
// k / kInitRoots, one per wave, and collects the distances 1 and 2 of the
// rows h < kInitHot in s_hot: bit k % kInitRoots of s_hot[h] is plane 1's
// bit, bit 16 + k % kInitRoots plane 2's.  plane_flush then writes them out.
// Bound by the atomics on the plane words: the top-ranked rows take a bit of
// nearly every root.  R-MAT-20, all batches: 17.8 ms with every entry an
// atomicOr, 13.6 with the hot rows collected here and flushed by atomicOr,
// 10.5 with plain 16-bit stores.
constexpr uint32_t kInitHot = 8192;
constexpr uint32_t kInitRoots = 16;

template <bool PLANES = false, bool HOT = false>
__device__ inline void phase_batch_init(const BuildArgs& A, const Exec& X, uint32_t ib, uint32_t bs, uint32_t bstamp,
                                        uint32_t* s_hot = nullptr) {
    const uint32_t lane = lane_id();
    for (uint32_t k = X.w; k < bs; k += X.nw) {
        const uint32_t u = ib + k;
        const uint32_t len = A.llen[u];
        const uint64_t off0 = A.loff[u];
        const uint32_t cap = A.lcap[u];
        // the first four chunks of L(u) and u's degree are loaded ahead of
        // the bookkeeping (a relocation by wave_reserve copies the same
        // entries, so they stay valid)
        uint32_t e[4];
#pragma unroll
        for (uint32_t c = 0; c < 4; ++c) {
            const uint32_t i = 64u * c + lane;
            e[c] = i < len ? A.arena[off0 + i] : 0u;
        }
        const uint64_t deg = A.rrow[u + 1] - A.rrow[u];
        const uint32_t tpos = shard_append(&X.qs[X.my].touched, lane == 0, (uint64_t)X.my * X.seg);
        if (lane == 0) {
            A.touch_stamp[u] = bstamp;
            A.touched[tpos] = u;
            A.tstart[tpos] = len;
        }
        if (A.bp_t && A.bp_used[u]) {  // a bit-parallel vertex is no root of the rounds
            if (lane == 0) A.act_v[0][k] = u;
            if (lane < A.W) A.act_delta[0][(size_t)k * A.W + lane] = 0ull;
            continue;
        }
        const uint64_t off = wave_reserve(A, X, u, off0, len, cap, 1);
        if (off == ~0ull) continue;
        const unsigned long long kq = 1ull << (k >> 4);
        if (lane == 0) {
            A.arena[off + len] = pll_pack(u, 0);
            A.llen[u] = len + 1;
            if (!PLANES) {
                A.T[(size_t)u * A.bstride + k] = 0;
                if (u >= A.hot) atomicOr((unsigned long long*)&A.rowmask[u], kq);
            }
        }
        // four chunks at a time: loaded before any is written out
        for (uint32_t i0 = 0; i0 < len; i0 += 256) {
            if (i0) {
#pragma unroll
                for (uint32_t c = 0; c < 4; ++c) {
                    const uint32_t i = i0 + 64u * c + lane;
                    e[c] = i < len ? A.arena[off + i] : 0u;
                }
            }
#pragma unroll
            for (uint32_t c = 0; c < 4; ++c) {
                if (i0 + 64u * c + lane < len) {
                    const uint32_t h = e[c] >> 8;
                    if (PLANES) {
                        const uint32_t d = e[c] & 255u;
                        if (HOT && d <= 2 && h < kInitHot)
                            atomicOr(&s_hot[h], (d == 1 ? 0x10001u : 0x10000u) << (k % kInitRoots));
                        else
                            plane_set(A, h, d, k);
                    } else {
                        A.T[(size_t)h * A.bstride + k] = (uint8_t)(e[c] & 255u);
                        if (h >= A.hot) atomicOr((unsigned long long*)&A.rowmask[h], kq);
                    }
                }
            }
        }
        if (lane == 0) A.act_v[0][k] = u;
        if (lane == 0 && A.act_rng[0]) A.act_rng[0][k] = make_uint2(len, 1u);  // the self entry
        if (lane < A.W) A.act_delta[0][(size_t)k * A.W + lane] = (lane == (k >> 6)) ? (1ull << (k & 63)) : 0ull;
        enqueue_heavy(A, X, 0, k, deg);
    }
}

// Write the workgroup's s_hot rows (below the batch's end: no other vertex is
// a hub yet) into planes 1 and 2; k0 is its first root's index in the batch.
// The top-ranked rows hold a bit of nearly every root, and atomics on one
// address serialise.  No other workgroup writes these 16 bits of a row's
// word, so they go out as plain 16-bit stores.
__device__ inline void plane_flush(const BuildArgs& A, uint32_t k0, uint32_t rows, const uint32_t* s_hot) {
    uint16_t* half = reinterpret_cast<uint16_t*>(A.P) + k0 / kInitRoots;
    for (uint32_t h = threadIdx.x; h < min(rows, kInitHot); h += blockDim.x) {
        const uint32_t x = s_hot[h];
        if (!x) continue;
        uint16_t* row = half + (size_t)h * (PLL_PLANES * 4u * A.W);
        if (x & 0xFFFFu) row[0] = (uint16_t)x;
        row[4u * A.W] = (uint16_t)(x >> 16);
    }
}

// The lanes with `enq` append r to receiver queue rq stored in recv, and of
// them those with `first` (r's first touch in this batch) to the touched
// list, with L(r)'s length tlen.  The whole wave calls it.  The two counters'
// atomics are issued together, so a call waits for one round trip.
__device__ inline void append_receivers(const BuildArgs& A, const Exec& X, uint32_t* recv, uint32_t rq, uint32_t r,
                                        bool enq, bool first, uint32_t tlen) {
    const uint64_t be = ballot64(enq), bf = ballot64(first);
    if (!be) return;
    const uint32_t lane = lane_id();
    const uint32_t leader = (uint32_t)__builtin_ctzll(be);
    uint32_t rb = 0, tb = 0;
    if (lane == leader) {
        rb = atomicAdd(&X.qs[X.my].recv[rq], (uint32_t)__builtin_popcountll(be));
        if (bf) tb = atomicAdd(&X.qs[X.my].touched, (uint32_t)__builtin_popcountll(bf));
    }
    const size_t seg = (size_t)X.my * X.seg;
    rb = readlane32(rb, leader);
    tb = readlane32(tb, leader);
    if (enq) recv[seg + rb + __builtin_popcountll(be & lanemask_lt())] = r;
    if (first) {
        const size_t tp = seg + tb + __builtin_popcountll(bf & lanemask_lt());
        A.touched[tp] = r;
        A.tstart[tp] = tlen;
    }
}

// The lanes whose vertex r got a delivery (`any`) take r's receiver slot
// of the next round (one per vertex and round, via its round stamp) into
// queue rq stored in recv; the lane that wins the slot also records r's
// first touch in this batch.  The whole wave calls it.
__device__ inline void enqueue_receivers(const BuildArgs& A, const Exec& X, uint32_t* recv, uint32_t rq,
                                         uint32_t rstamp, uint32_t bstamp, uint32_t r, bool any) {
    bool enq = false;
    uint32_t ts = bstamp, tlen = 0;
    if (any && A.recv_stamp[r] != rstamp) {
        // the winner's other reads fly with the exchange
        ts = A.touch_stamp[r];
        tlen = A.llen[r];
        enq = atomicExch(&A.recv_stamp[r], rstamp) != rstamp;
    }
    const bool first = enq && ts != bstamp;
    if (first) A.touch_stamp[r] = bstamp;
    append_receivers(A, X, recv, rq, r, enq, first, tlen);
}

// Deliver to vertex r the words w[k] of a delta whose candidates ranked
// above r are m[k] (0 for unused slots): each is filtered by C(r) and ORed
// into msgs(r).  The four C loads are issued before any is used, so the
// words of one edge cost one round trip.  Returns whether anything was
// delivered.
__device__ inline bool deliver4(const BuildArgs& A, uint64_t* msgs, uint32_t r, const uint32_t (&w)[4],
                                const uint64_t (&m)[4], bool filter) {
    uint64_t c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k] = filter && m[k] ? A.C[(size_t)r * A.W + w[k]] : 0ull;
    bool any = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint64_t x = m[k] & ~c[k];
        if (x) {
            atomicOr((unsigned long long*)&msgs[(size_t)r * A.W + w[k]], (unsigned long long)x);
            any = true;
        }
    }
    return any;
}

// Push delta L(a) (lane w < W holds word w in dl; nz marks the nonzero
// words) along the CSR entries [beg, end) of the active vertex a, into the
// message buffer msgs and receiver queue rq (counters) stored in recv.
// The next 64 neighbours load while this step delivers; first0 is the first
// step's, lane l's entry beg + l (0 past the end).  Without `filter` C(r) is
// not read (a batch's first push: it is empty).
__device__ inline void push_edges(const BuildArgs& A, const Exec& X, uint64_t* msgs, uint32_t* recv, uint32_t ib,
                                  uint32_t rq, uint32_t rstamp, uint32_t bstamp, uint64_t dl, uint64_t nz,
                                  uint64_t beg, uint64_t end, uint32_t first0, bool filter) {
    const uint32_t lane = lane_id();
    uint32_t next = first0;
    for (uint64_t e0 = beg; e0 < end; e0 += 64) {
        const uint64_t e = e0 + lane;
        const uint32_t r = next;
        next = e + 64 < end ? A.rcol[e + 64] : 0u;
        const bool fwd = e < end && r > ib;
        const uint32_t rel = r - ib;
        bool any = false;
        uint64_t todo = nz;
        while (todo) {  // four words at a time
            uint32_t w[4];
            uint64_t m[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                w[k] = todo ? (uint32_t)__builtin_ctzll(todo) : 0u;
                m[k] = todo && fwd ? readlane64(dl, w[k]) & rank_mask(rel, w[k]) : 0ull;
                todo &= todo - 1;
            }
            any |= deliver4(A, msgs, r, w, m, filter);
        }
        enqueue_receivers(A, X, recv, rq, rstamp, bstamp, r, any);
    }
}

// The heavy-row items of active list p, spread over every wave: pushes
// into msgs and receiver queue rq stored in recv.
__device__ inline void phase_push_heavy(const BuildArgs& A, const Exec& X, uint32_t ib, uint32_t p, uint32_t rq,
                                        uint64_t* msgs, uint32_t* recv, uint32_t rstamp, uint32_t bstamp,
                                        PhaseStats& st, bool filter) {
    const uint32_t lane = lane_id();
    const uint32_t* act_v = A.act_v[p];
    const uint64_t* act_d = A.act_delta[p];
    uint32_t pre;
    const uint32_t nh = shard_prefix(lane < X.nq ? X.qs[lane].hq[p] : 0u, pre);
    for (uint32_t t = X.w; t < nh; t += X.nw) {
        const uint32_t s = shard_of(X.nq, pre, t);
        const uint2 item = A.hq[p][s * A.hq_seg + (t - readlane32(pre, s))];
        const uint64_t dl = lane < A.W ? act_d[(size_t)item.x * A.W + lane] : 0ull;
        const uint64_t nz = ballot64(dl != 0);
        const uint32_t a = act_v[item.x];
        const uint64_t beg = A.rrow[a] + (uint64_t)item.y * kHeavyItem;
        const uint64_t end = min(A.rrow[a + 1], beg + kHeavyItem);
        if (lane == 0) st.edges += end - beg;
        push_edges(A, X, msgs, recv, ib, rq, rstamp, bstamp, dl, nz, beg, end,
                   beg + lane < end ? A.rcol[beg + lane] : 0u, filter);
    }
}

// Where a fused check takes its round from (message buffer and receiver
// list) and delivers the next one: that round's message buffer, receiver
// queue and counters, the round stamps, and whether it is pulled.
struct NextRound {
    uint64_t* msgs_in;
    uint32_t* recv_in;
    uint64_t* msgs;
    uint32_t* recv;
    uint32_t rin, rout, rclr, hout;
    uint32_t rstamp, bstamp;
    uint32_t pull;  // the next round is pulled (phase_pull4) instead of pushed
};

// A pulled round (the direction-optimizing alternative to push_edges, for
// rounds whose active vertices cover much of the graph): every vertex
// r > ib ORs the deltas of its active neighbours (act_at carries this
// round's stamp) and delivers the result exactly as the pushes from those
// neighbours would: masked to candidates ranked above r and not yet in
// C(r), into msgs(r), with one receiver slot and the first-touch record.
// Items are (vertex, segment of kPullSeg CSR entries); the segments of one
// vertex merge through atomicOr and the receiver stamp, like pushes do.
constexpr uint32_t kPullSeg = 256;

// A wave takes four items: the 16-lane group g = lane / 16
// gathers item i0 + g, 16 CSR entries at a time, and its lane 16g + w holds
// word w of the delta it collects.  Each step, every group ORs in the deltas
// of up to four of its active neighbours (the groups' steps run side by
// side), so sixteen delta lines are in flight in one wave; one neighbour per
// step made the gather a chain of one access per active neighbour (R-MAT-20
// 511 -> 393 us per gather, R-MAT-16 51 -> 31 us).
__device__ inline void phase_pull4(const BuildArgs& A, const Exec& X, uint32_t ib, const uint2* items,
                                   const uint32_t* nitems, uint32_t q, const NextRound& nr) {
    const uint32_t lane = lane_id();
    const uint32_t W = A.W;
    const uint32_t wd = lane & 15u, gsh = lane & 48u;
    const uint64_t* act_d = A.act_delta[q];
    const uint32_t total = *nitems;
    for (uint32_t t0 = 4u * X.w; t0 < total; t0 += 4u * X.nw) {
        const uint32_t t = t0 + (lane >> 4);
        const uint2 it = t < total ? items[t] : make_uint2(0u, 0u);
        const uint32_t r = it.x;
        const bool valid = t < total && r > ib;
        uint64_t beg = 0, end = 0;
        if (valid) {
            beg = A.rrow[r] + (uint64_t)it.y * kPullSeg;
            end = min(A.rrow[r + 1], beg + kPullSeg);
        }
        uint64_t m = 0;
        // a chunk's stamps load while the chunk before it is gathered, its
        // neighbours another chunk earlier
        const uint32_t deg = (uint32_t)(end - beg);
        const uint32_t* row = A.rcol + beg;
        uint64_t at = wd < deg ? A.act_at[row[wd]] : 0ull;
        uint32_t next = wd + 16u < deg ? row[wd + 16u] : 0u;
        for (uint32_t e0 = 0; ballot64(e0 < deg); e0 += 16) {
            const uint32_t e = e0 + wd;
            const uint64_t at1 = e + 16u < deg ? A.act_at[next] : 0ull;
            next = e + 32u < deg ? row[e + 32u] : 0u;
            const uint64_t am = ballot64(e < deg && (uint32_t)(at >> 32) == nr.rstamp);
            uint32_t gm = (uint32_t)(am >> gsh) & 0xFFFFu;  // this group's active neighbours
            while (ballot64(gm != 0)) {
                uint64_t d[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t l = gsh + (gm ? (uint32_t)__builtin_ctz(gm) : 0u);
                    const uint32_t slot = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(l * 4u), (int)(uint32_t)at);
                    d[k] = gm && wd < W ? act_d[(size_t)slot * W + wd] : 0ull;
                    gm &= gm - 1u;
                }
                m |= (d[0] | d[1]) | (d[2] | d[3]);
            }
            at = at1;
        }
        if (valid && wd < W) {
            m &= rank_mask(r - ib, wd);
            if (m) m &= ~A.C[(size_t)r * W + wd];
        } else {
            m = 0;
        }
        if (m) atomicOr((unsigned long long*)&nr.msgs[(size_t)r * W + wd], (unsigned long long)m);
        const uint64_t got = ballot64(m != 0);
        if (!got) continue;
        // one receiver slot per vertex and round, taken by lane 0 of the group
        enqueue_receivers(A, X, nr.recv, nr.rout, nr.rstamp, nr.bstamp, r, wd == 0 && ((got >> gsh) & 0xFFFFull) != 0);
    }
}

// The pull items of a rank-space CSR: (r, c) for every segment c of
// kPullSeg entries of every vertex r with neighbours, appended in any order.
__device__ inline void phase_pull_items(const BuildArgs& A, const Exec& X, uint2* items, uint32_t* nitems) {
    const uint32_t lane = lane_id();
    for (uint32_t r0 = X.w * 64u; r0 < A.n; r0 += X.nw * 64u) {
        const uint32_t r = r0 + lane;
        const uint64_t deg = r < A.n ? A.rrow[r + 1] - A.rrow[r] : 0ull;
        const uint32_t cnt = (uint32_t)((deg + kPullSeg - 1) / kPullSeg);
        const uint32_t pos = wave_excl_scan32(cnt);
        const uint32_t tot = readlane32(pos + cnt, 63);
        uint32_t base = 0;
        if (lane == 0 && tot) base = atomicAdd(nitems, tot);
        base = readlane32(base, 0);
        for (uint32_t c = 0; c < cnt; ++c) items[base + pos + c] = make_uint2(r, c);
    }
}

// Scatter phase of Algorithm 4 over active list p (nact slots) into msgs and
// receiver queue p stored in recv.
// Batch vertex u_k may be sent to v only when u_k outranks v (rank ib + k
// < v) and C(v) does not hold it yet.  Slots whose delta is empty are
// skipped; rows longer than kHeavy were queued as items and are spread over
// every wave after the per-slot pass.
__device__ inline void phase_push(const BuildArgs& A, const Exec& X, uint64_t* msgs, uint32_t* recv, uint32_t ib,
                                  uint32_t p, uint32_t nact, uint32_t rstamp, uint32_t bstamp, PhaseStats& st,
                                  bool filter) {
    const uint32_t lane = lane_id();
    if (X.zero_i < X.nq) X.qs[X.zero_i].hq[p ^ 1u] = 0;
    const uint32_t* act_v = A.act_v[p];
    const uint64_t* act_d = A.act_delta[p];
    for (uint32_t i = X.w; i < nact; i += X.nw) {
        const uint64_t dl = lane < A.W ? act_d[(size_t)i * A.W + lane] : 0ull;
        const uint64_t nz = ballot64(dl != 0);
        if (!nz) continue;
        const uint32_t a = act_v[i];
        const uint64_t beg = A.rrow[a], end = A.rrow[a + 1];
        if (end - beg > kHeavy) continue;
        if (lane == 0) st.edges += end - beg;
        push_edges(A, X, msgs, recv, ib, p, rstamp, bstamp, dl, nz, beg, end,
                   beg + lane < end ? A.rcol[beg + lane] : 0u, filter);
    }
    phase_push_heavy(A, X, ib, p, p, msgs, recv, rstamp, bstamp, st, filter);
}

// Lane `src`'s x in every lane (the LDS crossbar; src may differ per lane).
__device__ inline uint64_t shfl64(uint64_t x, uint32_t src) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(src * 4u), (int)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(src * 4u), (int)(uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Bit-parallel bound (Section 5.2) of every candidate in `mine` at v for
// distance j: candidate u_k is pruned when, for some BP root i,
// d_i(u_k) + d_i(v) - c <= j, with c = 2 when the S^-1 sets of u_k and v
// meet, else 1 when S^-1 of one meets S^0 of the other, else 0.  Lane i
// (< bp_t) holds v's data of root i; lanes run over the candidates of one
// word at a time, reading the batch vertices' data from the transposed
// per-batch copy.  Returns, in lane w, the pruned bits of word w.
// Bound by the latency of a candidate's 17 bytes per root: the word loop is
// scalar and four candidates load side by side (R-MAT-16 with 16 roots, the
// fused checks of a build: 5.3 -> 3.8 ms).
template <int WM>
__device__ inline uint64_t bp_prune_words(const BuildArgs& A, uint32_t v, uint32_t ib, uint32_t j, uint64_t mine) {
    const uint32_t lane = lane_id();
    const uint32_t t = A.bp_t;
    uint32_t dv = PLL_INF8;
    ulonglong2 sv = make_ulonglong2(0ull, 0ull);
    if (lane < t) {
        dv = A.bp_dist[(size_t)v * t + lane];
        sv = A.bp_sets[(size_t)v * t + lane];
    }
    const uint64_t roots_v = ballot64(lane < t && dv != PLL_INF8);
    uint64_t out = 0;
    // few candidates: lanes over the BP roots, a few candidates at a time (a
    // candidate's data of all roots is one coalesced load); otherwise lanes over the
    // candidates of a word, one root at a time
    const uint32_t ncand = wave_sum32(lane < WM ? (uint32_t)__builtin_popcountll(mine) : 0u);
    // (scalar loops over the words that hold candidates: one copy of the code)
    uint64_t words = ballot64(lane < WM && mine != 0);
    const uint32_t nwords = (uint32_t)__builtin_popcountll(words);
    if (ncand < nwords * (uint32_t)__builtin_popcountll(roots_v)) {
        // rl lanes hold the roots, up to four candidates side by side
        const uint32_t rl = t <= 16 ? 16u : t <= 32 ? 32u : 64u;
        const uint32_t i = lane & (rl - 1u), slot = lane / rl, nb = PLL_WAVE / rl;
        const uint32_t dvi = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(i * 4u), (int)dv);
        const uint64_t v1 = shfl64(sv.x, i), v0 = shfl64(sv.y, i);
        const bool root = i < t && dvi != PLL_INF8;
        while (words) {
            const uint32_t w = (uint32_t)__builtin_ctzll(words);
            words &= words - 1;
            uint64_t m = readlane64(mine, w);
            while (m) {
                // the slot's candidate: the lowest bits of m in order
                uint64_t bits[4];
#pragma unroll
                for (uint32_t x = 0; x < 4; ++x) {
                    bits[x] = x < nb ? m & (0ull - m) : 0ull;
                    m ^= bits[x];
                }
                const uint64_t mybit = slot == 0 ? bits[0] : slot == 1 ? bits[1] : slot == 2 ? bits[2] : bits[3];
                uint32_t td = 0xFFFFFFFFu;
                if (root && mybit) {
                    const size_t at = (size_t)(ib + 64u * w + (uint32_t)__builtin_ctzll(mybit)) * t + i;
                    const uint32_t du = A.bp_dist[at];
                    if (du != PLL_INF8) {
                        // the sets decide only where the sum is j + 1 or j + 2
                        td = du + dvi;
                        if (td > j && td <= j + 2u) {
                            const ulonglong2 su = A.bp_sets[at];
                            if (su.x & v1) td -= 2;
                            else if ((su.x & v0) | (su.y & v1)) td -= 1;
                        }
                    }
                }
                const uint64_t pr = ballot64(td <= j);
                uint64_t cut = 0;
#pragma unroll
                for (uint32_t x = 0; x < 4; ++x)
                    if (x < nb && ((pr >> (x * rl)) & (rl == 64 ? ~0ull : (1ull << rl) - 1ull))) cut |= bits[x];
                if (lane == w) out |= cut;
            }
        }
        return out;
    }
    while (words) {
        const uint32_t w = (uint32_t)__builtin_ctzll(words);
        words &= words - 1;
        const uint64_t m = readlane64(mine, w);
        const bool cand = (m >> lane) & 1ull;
        const uint32_t kk = 64u * w + lane;
        uint32_t bound = 0xFFFFFFFFu;
        uint64_t todo = roots_v;
        while (todo) {
            const uint32_t i = (uint32_t)__builtin_ctzll(todo);
            todo &= todo - 1;
            const uint32_t dvi = readlane32(dv, i);
            const uint64_t v1 = readlane64(sv.x, i), v0 = readlane64(sv.y, i);
            if (cand) {
                const uint32_t du = A.bpb_dist[(size_t)i * A.bstride + kk];
                if (du != PLL_INF8 && bound > j && du + dvi <= j + 2u) {
                    uint32_t td = du + dvi;
                    if (td > j) {
                        const ulonglong2 su = A.bpb_sets[(size_t)i * A.bstride + kk];
                        if (su.x & v1) td -= 2;
                        else if ((su.x & v0) | (su.y & v1)) td -= 1;
                    }
                    bound = min(bound, td);
                }
            }
        }
        const uint64_t pr = ballot64(cand && bound <= j);
        if (lane == w) out = pr;
    }
    return out;
}

// OR over each 16-lane row by DPP row rotations: every lane of a row gets
// its row's OR (the whole wave must be active).
__device__ inline uint32_t row_or32_dpp(uint32_t x) {
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xf, 0xf, false);  // row_ror:1
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xf, 0xf, false);  // row_ror:2
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xf, 0xf, false);  // row_ror:4
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, false);  // row_ror:8
    return x;
}

__device__ inline uint64_t row_or64_dpp(uint64_t x) {
    return ((uint64_t)row_or32_dpp((uint32_t)(x >> 32)) << 32) | row_or32_dpp((uint32_t)x);
}


// x of the lane N below (mod 16) in each 16-lane row.
template <int N>
__device__ inline uint64_t row_ror64(uint64_t x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, 0x120 + N, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), 0x120 + N, 0xf, 0xf, false);
    return ((uint64_t)hi << 32) | lo;
}

// Lane e's x (e = 0..15, a constant) in every lane of its 16-lane row (DPP
// row_newbcast; the whole wave must be active).
template <int E>
__device__ inline uint32_t row_bcast32(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x150 + E, 0xf, 0xf, true);
}

// The word offsets of the table lines that a group's entries name, for the
// lane's own slot: line i (< WM) is entry slot * WM + i of the row, where
// slot = sub / WM (one slot, the whole row, at WM = 16).
template <int WM, int I = 0>
__device__ inline void plane_lines(uint32_t at, uint32_t first, uint32_t (&line)[WM]) {
    if constexpr (I < WM) {
        if constexpr (WM == 16)
            line[I] = row_bcast32<I>(at);
        else
            line[I] = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((first + I) * 4u), (int)at);
        plane_lines<WM, I + 1>(at, first, line);
    }
}

// The pruning test on the bit planes (BuildArgs::P), for rounds j <=
// PLL_PLANES + 1.  The 16-lane group g takes 16 entries at a time: lane
// 16g + i reads entry i, and the entry's plane line (W words, one 128-byte
// line at W = 16) is then read by the group's lanes together, word w by the
// lanes with sub % WM = w.  So an entry tests every candidate of the vertex
// with one coalesced read and no compare or reduction, and the 16 lines of
// a chunk are independent loads in flight at once: a chunk costs two
// dependent accesses, where the byte table (prune_scan, prune_scan4) makes
// a row-mask access and one pass of 64-byte segment reads, compares and
// lane reductions per live candidate word (7.5 of them per entry in the
// R-MAT-20 rounds 2 and 3).  Lanes whose word has no live candidate load
// nothing.  For W < 16 the row's lanes hold 16 / WM lines side by side.
// Bound by those two dependent accesses, then by the appends and pushes around
// the scan.  R-MAT-20 build: 192 ms on the byte table, 167 on the planes; all
// later steps together take its fused checks from 125.7 to 80.7 ms.
//
// SHARE: one receiver for the whole wave (its candidates in lanes w < W, and
// group g takes entries 16g .. 16g + 15 of each 64); otherwise each group
// has its own receiver, list and candidates (lane 16g + w).  The source is
// L(v) or, with `nbr` in round 2, the neighbour row (see prune_scan_nbrs).
// Returns the pruned candidates in the lanes that hold the words of cw.
template <int WM, bool SHARE>
__device__ inline uint64_t prune_planes(const BuildArgs& A, uint64_t off, uint32_t len, bool nbr, uint32_t lim,
                                        uint32_t j, uint64_t cw, PhaseStats& st) {
    constexpr uint32_t kStep = SHARE ? 64u : 16u;
    const uint32_t lane = lane_id();
    const uint32_t sub = lane & 15u;
    const uint32_t gsh = lane & 48u;  // 16 * group
    const uint32_t wd = sub & (uint32_t)(WM - 1);
    const uint32_t first = gsh + sub - wd;  // first lane of this lane's slot
    const uint32_t zero = (A.n - 1u) * (PLL_PLANES * A.W);
    const uint32_t* src = (nbr ? A.rcol : A.arena) + off;
    const uint64_t* words = A.Pchk + wd;
    if (SHARE || WM < 16) cw = shfl64(cw, (SHARE ? 0u : gsh) + wd);
    uint64_t pw = 0;
    uint32_t idx = SHARE ? lane : sub;
    uint32_t next = idx < len ? src[idx] : 0u;
    for (uint32_t base = 0;; base += kStep, idx += kStep) {
        const uint64_t live = cw & ~pw;
        const uint64_t lb = ballot64(live != 0 && base < len);
        if (!lb) break;
        // this group still scans: candidates live and entries left
        const bool on = ((lb >> gsh) & 0xFFFFull) != 0;
        bool ok = on && idx < len;
        st.read += ok;
        const uint32_t ent = next;
        next = on && idx + kStep < len ? src[idx + kStep] : 0u;
        uint32_t h = ent, t = 1u;  // the neighbour row: T[h][k] <= 2 - 1
        if (nbr) {
            ok = ok && h < lim;
        } else {
            h = ent >> 8;
            const uint32_t d = ent & 255u;
            ok = ok && d != 0 && d < j;
            t = j - d;
        }
        const uint32_t row = h * (PLL_PLANES * A.W);
        uint64_t hit = 0;
        // plane 1 or 2, then the exact planes 3..t
        for (uint32_t p = 2;;) {
            const uint64_t okb = ballot64(ok);
            if (okb) {
                uint32_t line[WM];
                plane_lines<WM>(ok ? row + (min(t, p) - 1u) * A.W : zero, first, line);
                if (live != 0 && on && ((okb >> gsh) & 0xFFFFull)) {
#pragma unroll
                    for (int i = 0; i < WM; ++i) hit |= words[line[i]];
                    if (!(wd & 1u)) st.table += (uint32_t)__builtin_popcountll((okb >> first) & ((1ull << WM) - 1ull));
                }
            }
            if (++p >= j) break;
            ok = ok && t >= p;
        }
        // the lines of the row's slots, and of the wave's groups, together
        if (WM <= 8) hit |= row_ror64<8>(hit);
        if (WM <= 4) hit |= row_ror64<4>(hit);
        if (WM <= 2) hit |= row_ror64<2>(hit);
        if (WM <= 1) hit |= row_ror64<1>(hit);
        if (SHARE) {
            hit |= shfl64(hit, lane ^ 16u);
            hit |= shfl64(hit, lane ^ 32u);
        }
        pw |= hit & live;
    }
    return pw;
}

// Gather phase of Algorithm 4 for round j: one wave per
// receiver.  Receiver i (in shard order) becomes slot i of the next active
// list (with an empty delta when nothing was accepted).
//
// BP (bit-parallel labels present) is a separate instantiation: the BP
// bound's registers would otherwise cost every build occupancy.
//
// FUSE: the wave of a receiver that accepted something also pushes its
// delta L for round j+1 right away (rows up to kHeavy; longer rows become
// heavy items for a separate launch), into the other message buffer nr->msgs
// and receiver queue nr->rout, whose entries go to nr->recv (this round's
// receivers are read from nr->recv_in, so the two lists never share storage).
// C(r) of a neighbour may not hold this round's arrivals yet when the push
// reads it, so the check filters its messages by C(v) itself.  Receiver
// counters rotate over three (this round's nr->rin = p, the next round's,
// and nr->rclr, cleared here); active lists and heavy items use parity
// nr->hout.

template <int WM, bool BP = false, bool FUSE = false, bool SMALLT = false, bool PLANES = false>
__device__ inline void phase_check(const BuildArgs& A, const Exec& X, uint32_t ib, uint32_t bs, uint32_t j, uint32_t p,
                                   bool relaxed, PhaseStats& st, const NextRound* nr = nullptr) {
    const uint32_t lane = lane_id();
    const uint32_t W = A.W;
    const uint32_t q = FUSE ? nr->hout : p ^ 1u;
    uint64_t* const msgs = FUSE ? nr->msgs_in : A.msgs;
    const uint32_t* const recv = FUSE ? nr->recv_in : A.recv;
    uint32_t pre;
    const uint32_t nrecv = shard_prefix(lane < X.nq ? X.qs[lane].recv[p] : 0u, pre);
    // clear the counts the next launch appends to
    if (X.zero_i < X.nq) {
        if (FUSE) {
            X.qs[X.zero_i].recv[nr->rclr] = 0;
            X.qs[X.zero_i].hq[q ^ 1u] = 0;
        } else {
            X.qs[X.zero_i].recv[q] = 0;
        }
    }
    for (uint32_t i = X.w; i < nrecv; i += X.nw) {
        const uint32_t s = shard_of(X.nq, pre, i);
        const uint32_t v = recv[(size_t)s * X.seg + (i - readlane32(pre, s))];
        uint64_t mine = 0;
        if (lane < W) {
            const size_t at = (size_t)v * W + lane;
            mine = msgs[at];
            msgs[at] = 0;
            if (FUSE) mine &= ~A.C[at];
            A.C[at] |= mine;
        }
        const uint32_t len = A.llen[v];
        uint64_t off = A.loff[v];
        const uint32_t cap = A.lcap[v];
        // the row is needed by the push and by round 2's scan; its first
        // entries load beside the list's
        const uint64_t rbeg = A.rrow[v], rend = A.rrow[v + 1];
        uint32_t nb0 = 0;
        if (FUSE && lane < rend - rbeg) nb0 = A.rcol[rbeg + lane];
        uint64_t scan = mine;
        if (BP) {
            const uint64_t bpp = bp_prune_words<WM>(A, v, ib, j, mine);
            st.bp += __builtin_popcountll(lane < W ? bpp : 0ull);
            scan &= ~bpp;
        }
        // Round 1 never prunes: only an entry at distance 0, the self entry
        // (v, 0), could cover a candidate at distance 1, through T[v][k] <= 1,
        // i.e. with v a hub of u_k; but a candidate u_k only reaches vertices
        // ranked below it, and L(u_k) holds only hubs ranked above u_k.
        uint64_t pw = 0;
        if (PLANES) {
            if (j > 1) {
                const bool nbr = j == 2 && A.nbr_hubs && rend - rbeg < len;
                pw = prune_planes<WM, true>(A, nbr ? rbeg : off, nbr ? (uint32_t)(rend - rbeg) : len, nbr,
                                            min(v, ib + bs), j, scan, st);
            }
        } else if (j == 2 && A.nbr_hubs && rend - rbeg < len)
            pw = prune_scan_nbrs<WM, SMALLT>(A, v, min(v, relaxed ? ib : ib + bs), scan, st);
        else if (j > 1)
            pw = prune_scan<WM, SMALLT>(A, off, len, j, scan, relaxed, ib, st);
        const uint64_t acc = lane < W ? (scan & ~pw) : 0ull;
        const uint32_t cnt = (uint32_t)__builtin_popcountll(acc);
        const uint32_t pos = wave_excl_scan32(cnt);
        const uint32_t total = readlane32(pos + cnt, 63);
        st.cand += __builtin_popcountll(mine);
        st.cost_pos += (unsigned long long)len * (uint32_t)__builtin_popcountll(acc);
        st.cost_neg += (unsigned long long)len * (uint32_t)__builtin_popcountll(mine & ~acc);
        // the active list: the fused rounds read a slot only for a vertex
        // that accepted (its heavy-row items and pulled rounds); the
        // unfused ones push from every slot
        if (!FUSE || total != 0) {
            if (lane == 0) A.act_v[q][i] = v;
            if (lane < W) A.act_delta[q][(size_t)i * W + lane] = acc;
        }
        if (total == 0) continue;
        if (j >= PLL_INF8) {
            if (lane == 0) atomicOr(&A.ctr->error, PLL_ERR_DIST);
            continue;
        }
        off = wave_reserve(A, X, v, off, len, cap, total);
        if (off == ~0ull) continue;
        if (lane == 0) st.acc += total;
        const bool in_batch = v - ib < bs;
        const uint64_t lt = lanemask_lt();
        uint64_t todo = ballot64(acc != 0);
        while (todo) {
            const uint32_t w = (uint32_t)__builtin_ctzll(todo);
            todo &= todo - 1;
            const uint64_t aw = readlane64(acc, w);
            const uint32_t pwos = readlane32(pos, w);
            if ((aw >> lane) & 1ull) {
                const uint32_t k = w * 64u + lane;
                A.arena[off + len + pwos + __builtin_popcountll(aw & lt)] = pll_pack(ib + k, j);
                if (in_batch) {
                    if (PLANES) {
                        plane_set(A, ib + k, j, v - ib);
                    } else {
                        A.T[(size_t)(ib + k) * A.bstride + (v - ib)] = (uint8_t)j;
                        if (ib + k >= A.hot)
                            atomicOr((unsigned long long*)&A.rowmask[ib + k], 1ull << ((v - ib) >> 4));
                    }
                }
            }
        }
        if (lane == 0) A.llen[v] = len + total;
        if (FUSE && nr->pull) {  // the receivers gather: record where delta L(v) is
            if (lane == 0) {
                A.act_at[v] = ((uint64_t)nr->rstamp << 32) | i;
                st.pulled += rend - rbeg;
            }
            continue;
        }
        if (FUSE && rend - rbeg <= kHeavy) {
            if (lane == 0) st.edges += rend - rbeg;
            push_edges(A, X, nr->msgs, nr->recv, ib, nr->rout, nr->rstamp, nr->bstamp, acc, ballot64(acc != 0), rbeg,
                       rend, nb0, true);
        } else {
            enqueue_heavy(A, X, q, i, rend - rbeg);
        }
    }
}

// The pruning scans of four receivers at once: group g = lane / 16 scans
// the list of its own receiver 16 entries at a time, and lane 16g + w holds
// word w (< W <= 16) of that receiver's candidates in cw.  The test is the
// one of prune_scan and prune_scan_nbrs, per group: the source is either
// L(v) (entries arena[off .. off+len)) or, with `nbr`, v's neighbour row
// (rcol[off .. off+len), hubs ranked below lim at distance 1).  Each chunk
// makes one pass per live candidate word of each group (the groups'
// passes run side by side), and each group OR-reduces its word's prunes
// within its 16-lane row.  A group stops after the chunk that leaves none
// of its candidates live, or at its list's end.  Returns, in lane 16g + w,
// the pruned candidates of word w of receiver g.
template <int WM, bool SMALLT>
__device__ inline uint64_t prune_scan4(const BuildArgs& A, uint64_t off, uint32_t len, bool nbr, uint32_t lim,
                                       uint32_t j, uint64_t cw, bool relaxed, uint32_t ib, PhaseStats& st) {
    const uint32_t lane = lane_id();
    const uint32_t sub = lane & 15u;
    const uint32_t gsh = lane & 48u;  // 16 * group
    const uint32_t* src = (nbr ? A.rcol : A.arena) + off;
    uint64_t pw = 0;
    uint32_t next = sub < len ? src[sub] : 0u;
    for (uint32_t base = 0;; base += 16) {
        const uint64_t live_lane = cw & ~pw;
        const uint64_t lb = ballot64(live_lane != 0);
        // this group still scans: candidates live and entries left
        const bool gon = ((lb >> gsh) & 0xFFFFull) != 0 && base < len;
        const uint64_t todo0 = ballot64(gon && live_lane != 0);
        if (!todo0) break;
        const uint32_t idx = base + sub;
        bool ok = gon && idx < len;
        st.read += ok;
        const uint32_t ent = next;
        next = gon && idx + 16 < len ? src[idx + 16] : 0u;
        uint32_t h, tt;
        if (nbr) {
            h = ent;
            ok = ok && h < lim;
            tt = seg_tt<SMALLT>(1u);  // T[h][k] <= 2 - 1
        } else {
            h = ent >> 8;
            const uint32_t d = ent & 255u;
            ok = ok && d < j;
            if (relaxed) ok = ok && h < ib;
            // at most 254, the largest finite table byte (see prune_scan)
            tt = ok ? seg_tt<SMALLT>(min(j - d, PLL_INF8 - 1u)) : 0u;
        }
        const uint64_t rm = ok ? A.rmchk[h] : 0ull;
        const uint8_t* row = A.Tchk + (size_t)(ok ? h : 0u) * A.bstride;
        uint64_t todo = todo0;
        while (todo) {
            const uint32_t gm = (uint32_t)(todo >> gsh) & 0xFFFFu;
            const bool act = gm != 0;
            const uint32_t w = act ? (uint32_t)__builtin_ctz(gm) : 0u;
            uint64_t m = 0;
            if (act && ((rm >> (4 * w)) & 15u)) {
                m = seg_le<SMALLT>(row + 64u * w, tt);
                st.table += 4;
            }
            // the lane that holds word w masks the group's OR with its live
            // candidates (the OR of masked words is the masked OR)
            const uint64_t red = row_or64_dpp(m);
            const bool here = act && sub == w;
            if (here) pw |= red & live_lane;
            todo &= ~ballot64(here);
        }
    }
    return pw;
}

// Inclusive prefix sum within each 16-lane row (DPP row shifts; lanes
// shifted in from outside the row add 0; the whole wave must be active).
__device__ inline uint32_t row_incl_scan32(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);  // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);  // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);  // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);  // row_shr:8
    return x;
}

// push_edges for up to four receivers of one wave at once: group g's delta
// words are in lanes 16g + w of acc4, and its row is rcol[beg .. beg + deg)
// (beg and deg held by the group's lanes; deg = 0 for a group that pushes
// nothing here).  The rows are walked as one concatenated range, 64 edges
// per step, each lane taking the delta of its edge's receiver; deliveries
// and receiver slots are those of push_edges.
__device__ inline void push_edges4(const BuildArgs& A, const Exec& X, const NextRound& nr, uint32_t ib, uint64_t acc4,
                                   uint64_t beg, uint32_t deg) {
    const uint32_t lane = lane_id();
    // starts of groups 1..3 in the concatenation, and its length
    const uint32_t s1 = readlane32(deg, 0);
    const uint32_t s2 = s1 + readlane32(deg, 16);
    const uint32_t s3 = s2 + readlane32(deg, 32);
    const uint32_t D = s3 + readlane32(deg, 48);
    const uint64_t b0 = readlane64(beg, 0), b1 = readlane64(beg, 16), b2 = readlane64(beg, 32),
                   b3 = readlane64(beg, 48);
    // bit 16g + w: group g has a delta in word w
    const uint64_t nzl = ballot64(acc4 != 0);
    for (uint32_t t0 = 0; t0 < D; t0 += 64) {
        const uint32_t t = t0 + lane;
        // the last group whose start is <= t (empty groups share the next one's start)
        const uint32_t gl = (uint32_t)(t >= s1) + (uint32_t)(t >= s2) + (uint32_t)(t >= s3);
        const uint64_t bg = gl == 0 ? b0 : gl == 1 ? b1 : gl == 2 ? b2 : b3;
        const uint32_t sg = gl == 0 ? 0u : gl == 1 ? s1 : gl == 2 ? s2 : s3;
        const bool in = t < D;
        const uint32_t r = in ? A.rcol[bg + (t - sg)] : 0u;
        const bool fwd = in && r > ib;
        const uint32_t rel = r - ib;
        bool any = false;
        // the nonzero words of this edge's receiver, four at a time
        uint32_t todo = fwd ? (uint32_t)(nzl >> (16u * gl)) & 0xFFFFu : 0u;
        while (ballot64(todo != 0)) {
            uint32_t w[4];
            uint64_t m[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                w[k] = todo ? (uint32_t)__builtin_ctz(todo) : 0u;
                const uint64_t x = shfl64(acc4, 16u * gl + w[k]);
                m[k] = todo ? x & rank_mask(rel, w[k]) : 0ull;
                todo &= todo - 1;
            }
            any |= deliver4(A, nr.msgs, r, w, m, true);
        }
        enqueue_receivers(A, X, nr.recv, nr.rout, nr.rstamp, nr.bstamp, r, any);
    }
}

// The fused check (FUSE of phase_check, without bit-parallel labels) with
// four receivers per wave: receivers i0 .. i0+3 are read and scanned side by
// side by the four 16-lane groups (prune_scan4), so four receivers' chains
// of dependent loads (receiver, list, label chunk, row mask, table segment)
// are in flight in one wave.  The accepted entries are then appended one
// receiver after another, and the next round's deliveries of all four go
// out in one pass over their concatenated rows (push_edges4).  Active-list
// slots, heavy rows, pulled rounds and statistics are phase_check's.
template <int WM, bool SMALLT, bool PLANES = false>
__device__ inline void phase_check4(const BuildArgs& A, const Exec& X, uint32_t ib, uint32_t bs, uint32_t j,
                                    bool relaxed, PhaseStats& st, const NextRound& nr) {
    const uint32_t lane = lane_id();
    const uint32_t W = A.W;
    const uint32_t sub = lane & 15u, g = lane >> 4;
    const uint32_t q = nr.hout;
    uint32_t pre;
    const uint32_t nrecv = shard_prefix(lane < X.nq ? X.qs[lane].recv[nr.rin] : 0u, pre);
    // clear the counts the next launch appends to
    if (X.zero_i < X.nq) {
        X.qs[X.zero_i].recv[nr.rclr] = 0;
        X.qs[X.zero_i].hq[q ^ 1u] = 0;
    }
    for (uint32_t i0 = 4u * X.w; i0 < nrecv; i0 += 4u * X.nw) {
        const uint32_t ng = min(4u, nrecv - i0);
        uint32_t slot = 0;
        for (uint32_t gg = 0; gg < ng; ++gg) {
            const uint32_t s = shard_of(X.nq, pre, i0 + gg);
            const uint32_t at = s * X.seg + (i0 + gg - readlane32(pre, s));
            if (g == gg) slot = at;
        }
        const bool has = g < ng;
        const uint32_t i = i0 + g;
        const uint32_t v = has ? nr.recv_in[slot] : 0u;
        uint64_t mine = 0;
        if (has && sub < W) {
            const size_t at = (size_t)v * W + sub;
            mine = nr.msgs_in[at];
            nr.msgs_in[at] = 0;
            mine &= ~A.C[at];
            A.C[at] |= mine;
        }
        const uint32_t len = has ? A.llen[v] : 0u;
        const uint64_t off = has ? A.loff[v] : 0ull;
        // round 1 never prunes (see phase_check); round 2 reads the
        // neighbour row when it is the shorter source
        uint64_t pw = 0;
        if (j > 1) {
            bool nbr = false;
            uint64_t soff = off;
            uint32_t slen = len, lim = 0;
            if (j == 2 && A.nbr_hubs && has) {
                const uint64_t rb = A.rrow[v], re = A.rrow[v + 1];
                if (re - rb < len) {
                    nbr = true;
                    soff = rb;
                    slen = (uint32_t)(re - rb);
                    lim = min(v, relaxed ? ib : ib + bs);
                }
            }
            if (PLANES)
                pw = prune_planes<WM, false>(A, soff, slen, nbr, lim, j, mine, st);
            else
                pw = prune_scan4<WM, SMALLT>(A, soff, slen, nbr, lim, j, mine, relaxed, ib, st);
        }
        const uint64_t acc4 = mine & ~pw;
        st.cand += __builtin_popcountll(mine);
        st.cost_pos += (unsigned long long)len * (uint32_t)__builtin_popcountll(acc4);
        st.cost_neg += (unsigned long long)len * (uint32_t)__builtin_popcountll(mine & ~acc4);
        const uint64_t accl = ballot64(acc4 != 0);
        if (!accl) continue;  // nothing accepted: no slots, no pushes
        const bool gacc = ((accl >> (lane & 48u)) & 0xFFFFull) != 0;
        if (gacc) {  // the active-list slot of a receiver that accepted
            if (sub == 0) A.act_v[q][i] = v;
            if (sub < W) A.act_delta[q][(size_t)i * W + sub] = acc4;
        }
        if (j >= PLL_INF8) {
            if (lane == 0) atomicOr(&A.ctr->error, PLL_ERR_DIST);
            continue;
        }
        // entries of each word before it, within each receiver's candidates
        const uint32_t incl = row_incl_scan32((uint32_t)__builtin_popcountll(acc4));
        uint32_t appended = 0;  // bit gg: receiver gg's entries are in its list
        for (uint32_t gg = 0; gg < ng; ++gg) {
            uint64_t todo = (accl >> (16u * gg)) & 0xFFFFull;
            if (!todo) continue;
            const uint32_t vg = readlane32(v, 16u * gg);
            const uint32_t lg = readlane32(len, 16u * gg);
            const uint32_t total = readlane32(incl, 16u * gg + 15u);
            const uint64_t og = wave_reserve(A, X, vg, readlane64(off, 16u * gg), lg, A.lcap[vg], total);
            if (og == ~0ull) continue;
            if (lane == 0) st.acc += total;
            const bool in_batch = vg - ib < bs;
            const uint64_t lt = lanemask_lt();
            while (todo) {
                const uint32_t w = (uint32_t)__builtin_ctzll(todo);
                todo &= todo - 1;
                const uint64_t aw = readlane64(acc4, 16u * gg + w);
                const uint32_t pwos = readlane32(incl, 16u * gg + w) - (uint32_t)__builtin_popcountll(aw);
                if ((aw >> lane) & 1ull) {
                    const uint32_t k = w * 64u + lane;
                    A.arena[og + lg + pwos + __builtin_popcountll(aw & lt)] = pll_pack(ib + k, j);
                    if (in_batch) {
                        if (PLANES) {
                            plane_set(A, ib + k, j, vg - ib);
                        } else {
                            A.T[(size_t)(ib + k) * A.bstride + (vg - ib)] = (uint8_t)j;
                            if (ib + k >= A.hot)
                                atomicOr((unsigned long long*)&A.rowmask[ib + k], 1ull << ((vg - ib) >> 4));
                        }
                    }
                }
            }
            if (lane == 0) A.llen[vg] = lg + total;
            appended |= 1u << gg;
        }
        // round j+1: pulled (record where delta L(v) is) or pushed along the
        // rows, those longer than kHeavy as heavy items of a separate launch
        const bool out = (appended >> g) & 1u;
        uint64_t rb = 0;
        uint32_t deg = 0;
        if (out) {
            rb = A.rrow[v];
            deg = (uint32_t)(A.rrow[v + 1] - rb);
        }
        if (nr.pull) {
            if (out && sub == 0) {
                A.act_at[v] = ((uint64_t)nr.rstamp << 32) | i;
                st.pulled += deg;
            }
            continue;
        }
        const bool heavy = deg > kHeavy;
        if (out && !heavy && sub == 0) st.edges += deg;
        uint64_t hv = ballot64(out && heavy && sub == 0);
        while (hv) {
            const uint32_t l = (uint32_t)__builtin_ctzll(hv);
            hv &= hv - 1;
            enqueue_heavy(A, X, q, i0 + l / 16u, readlane32(deg, l));
        }
        push_edges4(A, X, nr, ib, acc4, rb, out && !heavy ? deg : 0u);
    }
}

// Per byte: min(x + d, 255) with dd = d * 0x01010101.  The low 7 bits of
// each byte are added without carries leaving the byte; the carry out of
// bit 7 marks the bytes that saturate.
__device__ inline uint32_t add_sat4(uint32_t x, uint32_t dd) {
    const uint32_t H = 0x80808080u;
    const uint32_t low = (x & ~H) + (dd & ~H);
    const uint32_t sum = low ^ ((x ^ dd) & H);
    const uint32_t ovf = ((x & dd) | ((x | dd) & ~sum)) & H;
    return sum | ((ovf >> 7) * 0xFFu);
}

// Bit i: min(p[i] + d, 255) <= thr[i], for 64 consecutive table bytes p and
// thresholds thr (le4_flags compares bytes against any per-byte threshold).
__device__ inline uint64_t sum_le_mask64(const uint8_t* p, uint32_t dd, const uint4* thr) {
    const uint4* q = reinterpret_cast<const uint4*>(p);
    uint64_t m = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint4 v = q[i];
        const uint4 t = thr[i];
        const uint32_t b = gather16(le4_flags(add_sat4(v.x, dd), t.x), le4_flags(add_sat4(v.y, dd), t.y),
                                    le4_flags(add_sat4(v.z, dd), t.z), le4_flags(add_sat4(v.w, dd), t.w));
        m |= (uint64_t)b << (16 * i);
    }
    return m;
}

// prune_scan with a distance per candidate: s_thr (LDS, 64 * W bytes) holds
// D(v); candidate u_k is pruned when some entry (h, d) of the list has
// T[h][k] + d <= D(v)[k].  Lanes beyond the live candidates are masked off,
// so bytes of 255 (no candidate) never count.  RECHECK: the candidates are
// entries of the list themselves, and none counts as covered by its own hub
// (ib: the batch's first rank); s_top (LDS, W words) holds the largest
// distance in each candidate word.  A table entry other than a hub's own is
// at least 1, so an entry at distance d covers only candidates above d and
// is left out of the words that have none.  Bound by the dependent segment
// reads and the byte adds (VALU): the scan stops at the chunk that leaves no
// candidate live and makes one pass per live word.  Weighted R-MAT-16: checks
// 5.8 ms a build (34 us a round), batch ends 3.4 ms before s_top, 3.0 with it.
// Unweighted R-MAT-16 with the recheck, batch ends: one scan per distance 2.41
// ms and 156 M table quarters (of the build), one scan for all 3.90 ms and
// 674 M, with s_top 2.09 ms and 150 M; with the relaxed check 3.36, 8.13 and
// 4.30 ms.
template <int WM, bool RECHECK = false>
__device__ inline uint64_t prune_scan_w(const BuildArgs& A, uint64_t off, uint32_t len, uint64_t cw,
                                        const uint4* s_thr, uint32_t ib, PhaseStats& st,
                                        const uint32_t* s_top = nullptr) {
    const uint32_t lane = lane_id();
    uint64_t pw = 0;
    const uint32_t top = RECHECK && lane < A.W ? s_top[lane] : 0u;
    const uint32_t top_all = RECHECK ? wave_max32(top) : 0u;
    // one pass per word that still holds live candidates, its prunes reduced
    // at once, and the next chunk's entries loaded ahead, as in prune_scan
    uint32_t next = lane < len ? A.arena[off + lane] : 0u;
    for (uint32_t base = 0; base < len; base += 64) {
        const uint32_t idx = base + lane;
        const bool ok = idx < len;
        st.read += ok;
        const uint32_t ent = next;
        next = idx + 64 < len ? A.arena[off + idx + 64] : 0u;
        const uint32_t h = ent >> 8, d = ent & 255u;
        const uint64_t rm = ok && (!RECHECK || (d != 0 && d < top_all)) ? A.rmchk[h] : 0ull;
        const uint32_t dd = d * 0x01010101u;
        const uint8_t* row = A.Tchk + (size_t)h * A.bstride;
        const uint64_t live_lane = cw & ~pw;
        uint64_t lw = ballot64(live_lane != 0) & (WM >= 64 ? ~0ull : ((1ull << WM) - 1ull));
        while (lw) {
            const uint32_t w = (uint32_t)__builtin_ctzll(lw);
            lw &= lw - 1;
            uint64_t m = 0;
            const uint32_t top_w = readlane32(top, w);
            if (((rm >> (4 * w)) & 15u) && (!RECHECK || d < top_w)) {
                m = sum_le_mask64(row + 64u * w, dd, s_thr + 4 * w);
                st.table += 4;
                const uint32_t self = h - ib;
                if (RECHECK && self >> 6 == w) m &= ~(1ull << (self & 63u));
            }
            const uint64_t red = wave_or64_u(m);
            if (lane == w) pw |= red & live_lane;
        }
        if (!ballot64((cw & ~pw) != 0)) break;
    }
    return pw;
}

// Write the batch entries (u_k, s_dist[k]) of the hubs k set in s_pres (W
// words) to the arena from `at` on, in ascending hub rank; returns how many.
__device__ inline uint32_t segment_emit(const BuildArgs& A, uint32_t ib, uint64_t at, const uint64_t* s_pres,
                                        const uint8_t* s_dist) {
    const uint32_t lane = lane_id();
    const uint64_t pw = lane < A.W ? s_pres[lane] : 0ull;
    const uint32_t cnt = (uint32_t)__builtin_popcountll(pw);
    const uint32_t pos = wave_excl_scan32(cnt);
    const uint32_t total = readlane32(pos + cnt, 63);
    uint64_t todo = ballot64(pw != 0);
    while (todo) {
        const uint32_t w = (uint32_t)__builtin_ctzll(todo);
        todo &= todo - 1;
        const uint64_t aw = readlane64(pw, w);
        const uint32_t base = readlane32(pos, w);
        if ((aw >> lane) & 1ull) {
            const uint32_t k = w * 64u + lane;
            A.arena[at + base + __builtin_popcountll(aw & lanemask_lt())] = pll_pack(ib + k, s_dist[k]);
        }
    }
    return total;
}

// Batch end, one wave per touched vertex v: clear C(v); sort the
// entries this batch appended to L(v) by hub rank; with `recheck`, first
// drop every such entry (u, d) that L(u) and L(v) already cover through
// another hub at distance <= d (Section 5.1's recheck with the batch's
// tables still in memory).  s_pres and s_top (W words each) and s_dist (b
// bytes) are this wave's LDS scratch.
//
// Weighted graphs (WEIGHTED): the recheck always runs (it is what makes the
// labels canonical there), D(v) is reset instead of C(v), and a hub may
// appear several times in the batch segment, each later entry shorter than
// the one before; only the last one is kept (s_pos, b words of LDS, holds
// the position of each hub's last entry).
template <int WM, bool WEIGHTED = false>
__device__ inline void phase_batch_end(const BuildArgs& A, const Exec& X, uint32_t ib, uint32_t bs, bool recheck,
                                       uint64_t* s_pres, uint32_t* s_top, uint8_t* s_dist, uint32_t* s_pos,
                                       PhaseStats& st) {
    const uint32_t lane = lane_id();
    const uint32_t W = A.W;
    if (WEIGHTED) recheck = true;
    uint32_t pre;
    const uint32_t ntouched = shard_prefix(lane < X.nq ? X.qs[lane].touched : 0u, pre);
    for (uint32_t i = X.w; i < ntouched; i += X.nw) {
        const uint32_t sh = shard_of(X.nq, pre, i);
        const size_t at = (size_t)sh * X.seg + (i - readlane32(pre, sh));
        const uint32_t v = A.touched[at];
        const uint32_t ts = A.tstart[at];
        const uint32_t len = A.llen[v];
        const uint64_t off = A.loff[v];
        if (WEIGHTED) {
            uint4* drow = reinterpret_cast<uint4*>(A.D + (size_t)v * A.bstride);
            for (uint32_t c = lane; c < 4 * W; c += 64) drow[c] = make_uint4(~0u, ~0u, ~0u, ~0u);
        } else if (lane < W) {
            A.C[(size_t)v * W + lane] = 0;
        }
        const uint32_t tail = len - ts;
        if (tail < 2 && !(recheck && tail >= 1)) continue;
        // A segment appended in one round is already in ascending hub rank
        // (each acceptance appends its candidates in ascending order): without
        // the recheck, a segment of up to 64 entries that is sorted stays.
        if (!recheck && tail <= 64) {
            const uint32_t e = lane < tail ? A.arena[off + ts + lane] : ~0u;
            const uint32_t nx = (uint32_t)__shfl_down((int)e, 1, 64);
            if (!ballot64(lane + 1 < tail && e >= nx)) continue;
        }
        if (lane < W) {
            s_pres[lane] = 0;
            s_top[lane] = 0;
        }
        if (WEIGHTED) {
            for (uint32_t k = lane; k < bs; k += 64) s_pos[k] = 0;
            wave_lds_sync();
            for (uint32_t x = ts + lane; x < len; x += 64) atomicMax(&s_pos[(A.arena[off + x] >> 8) - ib], x - ts + 1);
        }
        wave_lds_sync();
        for (uint32_t x = ts + lane; x < len; x += 64) {
            const uint32_t e = A.arena[off + x];
            const uint32_t k = (e >> 8) - ib;
            if (WEIGHTED && s_pos[k] != x - ts + 1) continue;
            s_dist[k] = (uint8_t)(e & 255u);
            if (recheck) atomicMax(&s_top[k >> 6], e & 255u);
            atomicOr((unsigned long long*)&s_pres[k >> 6], 1ull << (k & 63));
        }
        wave_lds_sync();
        if (recheck) {
            // one scan for all entries, each at its own distance.  No order
            // among them matters: a canonical entry is never covered by
            // another hub, and every other one is by a canonical hub.
            const bool in_batch = v - ib < bs;
            const uint64_t pr = prune_scan_w<WM, true>(A, off, len, lane < W ? s_pres[lane] : 0ull,
                                                       reinterpret_cast<const uint4*>(s_dist), ib, st, s_top);
            if (lane < W && pr) s_pres[lane] &= ~pr;
            st.removed += __builtin_popcountll(pr);
            if (in_batch) {
                uint64_t todo = ballot64(pr != 0);
                while (todo) {
                    const uint32_t w = (uint32_t)__builtin_ctzll(todo);
                    todo &= todo - 1;
                    if ((readlane64(pr, w) >> lane) & 1ull)
                        A.T[(size_t)(ib + w * 64u + lane) * A.bstride + (v - ib)] = (uint8_t)PLL_INF8;
                }
            }
            wave_lds_sync();
        }
        // emit the batch segment in ascending hub rank
        const uint32_t total = segment_emit(A, ib, off + ts, s_pres, s_dist);
        if (lane == 0 && total != tail) A.llen[v] = ts + total;
        wave_lds_sync();
    }
}

// The position of this lane's x among its 16-lane row's (distinct) values.
template <int N = 1>
__device__ inline uint32_t row_rank32(uint32_t x) {
    if constexpr (N < 16) {
        const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x120 + N, 0xf, 0xf, false);  // row_ror:N
        return (y < x ? 1u : 0u) + row_rank32<N + 1>(x);
    }
    return 0u;
}

// The batch end of an unweighted build without the recheck, four touched
// vertices per wave, one per 16-lane group: the batches of a large graph
// touch hundreds of thousands of vertices and append fewer than 16 entries
// to most, and one vertex per wave left 48 lanes idle behind a chain of
// dependent reads.  A segment of up to 16 entries is sorted in registers
// (each entry's position is the number of smaller ones in its row); longer
// ones take the whole wave, one after another, through the presence bitmap
// of phase_batch_end.  Bound by the chain of dependent reads and the C rows'
// clearing (128 bytes per vertex).  R-MAT-20, all batches: 12.9 ms one vertex
// per wave, 6.6 so; the build 157 -> 153.7 ms.
__device__ inline void phase_batch_end4(const BuildArgs& A, const Exec& X, uint32_t ib, uint64_t* s_pres,
                                        uint8_t* s_dist) {
    const uint32_t lane = lane_id();
    const uint32_t W = A.W;
    const uint32_t sub = lane & 15u, g = lane >> 4;
    uint32_t pre;
    const uint32_t ntouched = shard_prefix(lane < X.nq ? X.qs[lane].touched : 0u, pre);
    for (uint32_t i0 = 4u * X.w; i0 < ntouched; i0 += 4u * X.nw) {
        const uint32_t ng = min(4u, ntouched - i0);
        size_t at = 0;
        for (uint32_t gg = 0; gg < ng; ++gg) {
            const uint32_t sh = shard_of(X.nq, pre, i0 + gg);
            const size_t x = (size_t)sh * X.seg + (i0 + gg - readlane32(pre, sh));
            if (g == gg) at = x;
        }
        const bool has = g < ng;
        const uint32_t v = has ? A.touched[at] : 0u;
        const uint32_t ts = has ? A.tstart[at] : 0u;
        const uint32_t len = has ? A.llen[v] : 0u;
        const uint64_t seg = (has ? A.loff[v] : 0ull) + ts;
        if (has && sub < W) A.C[(size_t)v * W + sub] = 0;
        const uint32_t tail = len - ts;
        const bool here = tail >= 2u && tail <= 16u && sub < tail;
        const uint32_t e = here ? A.arena[seg + sub] : ~0u - sub;  // distinct, above every entry
        const uint32_t pos = row_rank32(e);
        if (here && pos != sub) A.arena[seg + pos] = e;
        uint64_t longer = ballot64(sub == 0 && tail > 16u);
        while (longer) {
            const uint32_t l = (uint32_t)__builtin_ctzll(longer);
            longer &= longer - 1;
            const uint32_t tg = readlane32(tail, l);
            const uint32_t* ent = A.arena + readlane64(seg, l);
            if (tg <= 64) {  // one round's entries are in order already
                const uint32_t x = lane < tg ? ent[lane] : ~0u;
                const uint32_t nx = (uint32_t)__shfl_down((int)x, 1, 64);
                if (!ballot64(lane + 1 < tg && x >= nx)) continue;
            }
            if (lane < W) s_pres[lane] = 0;
            wave_lds_sync();
            for (uint32_t x = lane; x < tg; x += 64) {
                const uint32_t k = (ent[x] >> 8) - ib;
                s_dist[k] = (uint8_t)(ent[x] & 255u);
                atomicOr((unsigned long long*)&s_pres[k >> 6], 1ull << (k & 63));
            }
            wave_lds_sync();
            segment_emit(A, ib, readlane64(seg, l), s_pres, s_dist);
            wave_lds_sync();
        }
    }
}

// ---- weighted graphs (Section 5.1) ----------------------------------------------------------------
//
// A candidate now carries its own distance d + w_e, and a round no longer
// equals a distance: a candidate can come back shorter in a later round.
// D(v) replaces C(v) as the filter (a candidate passes only if it lowers
// D(v)[k]); the pruning check compares each candidate with its own
// distance; a vertex that accepts pushes the entries it accepted (its
// delta L) rather than a bit-vector.  Entries accepted on the way may be
// non-canonical; the batch-end recheck removes them.

// D[p] = min(D[p], nd) on one byte (a compare-and-swap on its aligned word);
// true when this call lowered it.
__device__ inline bool byte_atomic_min(uint8_t* p, uint32_t nd) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(p);
    uint32_t* wp = reinterpret_cast<uint32_t*>(a & ~uintptr_t(3));
    const uint32_t sh = (uint32_t)(a & 3u) * 8u;
    uint32_t old = __hip_atomic_load(wp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (;;) {
        if (nd >= ((old >> sh) & 255u)) return false;
        const uint32_t nw = (old & ~(255u << sh)) | (nd << sh);
        const uint32_t prev = atomicCAS(wp, old, nw);
        if (prev == old) return true;
        old = prev;
    }
}

// Push the cnt entries at arena[eoff ..] (what the active vertex accepted
// last round) along its weighted CSR entries [beg, end).
__device__ inline void push_edges_w(const BuildArgs& A, const Exec& X, uint32_t ib, uint32_t p, uint32_t rstamp,
                                    uint32_t bstamp, uint64_t eoff, uint32_t cnt, uint64_t beg, uint64_t end) {
    const uint32_t lane = lane_id();
    for (uint64_t e0 = beg; e0 < end; e0 += 64) {
        const uint64_t e = e0 + lane;
        const bool in = e < end;
        const uint32_t r = in ? A.rcol[e] : 0u;
        const uint32_t wt = in ? A.rw[e] : 0u;
        const bool cand = in && r > ib;
        bool any = false, over = false;
        if (ballot64(cand)) {
            for (uint32_t t = 0; t < cnt; ++t) {
                const uint32_t ent = A.arena[eoff + t];
                const uint32_t k = (ent >> 8) - ib;
                const uint32_t nd = (ent & 255u) + wt;
                if (cand && r - ib > k) {  // only to vertices ranked below u_k
                    uint8_t* pd = A.D + (size_t)r * A.bstride + k;
                    if (nd >= PLL_INF8) {
                        // too long for the labels; harmless when a shorter
                        // candidate already reached r, else the build fails
                        over = over || *pd == PLL_INF8;
                    } else {
                        if (nd < *pd && byte_atomic_min(pd, nd)) {
                            atomicOr((unsigned long long*)&A.msgs[(size_t)r * A.W + (k >> 6)],
                                     (unsigned long long)(1ull << (k & 63)));
                            any = true;
                        }
                    }
                }
            }
        }
        if (ballot64(over) && lane == 0) atomicOr(&A.ctr->error, PLL_ERR_DIST);
        enqueue_receivers(A, X, A.recv, p, rstamp, bstamp, r, any);
    }
}

// Scatter phase for weighted graphs over active list p.
__device__ inline void phase_push_w(const BuildArgs& A, const Exec& X, uint32_t ib, uint32_t p, uint32_t nact,
                                    uint32_t rstamp, uint32_t bstamp, PhaseStats& st) {
    const uint32_t lane = lane_id();
    if (X.zero_i < X.nq) X.qs[X.zero_i].hq[p ^ 1u] = 0;
    for (uint32_t i = X.w; i < nact; i += X.nw) {
        const uint2 rg = A.act_rng[p][i];
        if (rg.y == 0) continue;
        const uint32_t a = A.act_v[p][i];
        const uint64_t beg = A.rrow[a], end = A.rrow[a + 1];
        if (end - beg > kHeavy) continue;
        if (lane == 0) st.edges += end - beg;
        push_edges_w(A, X, ib, p, rstamp, bstamp, A.loff[a] + rg.x, rg.y, beg, end);
    }
    uint32_t pre;
    const uint32_t nh = shard_prefix(lane < X.nq ? X.qs[lane].hq[p] : 0u, pre);
    for (uint32_t t = X.w; t < nh; t += X.nw) {
        const uint32_t s = shard_of(X.nq, pre, t);
        const uint2 item = A.hq[p][s * A.hq_seg + (t - readlane32(pre, s))];
        const uint2 rg = A.act_rng[p][item.x];
        const uint32_t a = A.act_v[p][item.x];
        const uint64_t beg = A.rrow[a] + (uint64_t)item.y * kHeavyItem;
        const uint64_t end = min(A.rrow[a + 1], beg + kHeavyItem);
        if (lane == 0) st.edges += end - beg;
        push_edges_w(A, X, ib, p, rstamp, bstamp, A.loff[a] + rg.x, rg.y, beg, end);
    }
}

// A pulled round for weighted graphs: one wave per (vertex r > ib, segment of
// kPullSeg CSR entries) of `items`.  It collects the smallest candidate
// distance of every root in LDS (s_min, b words) from the entries that r's
// active neighbours accepted last round (act_at carries that round's stamp),
// then lowers D(r) and sets the message bits where that is shorter than
// D(r): the same D, messages and receivers as push_edges_w's byte minima.
// The pushes are bound by those minima (a read, a compare-and-swap and an OR
// at scattered addresses per edge and entry); here an entry of an edge costs
// a coalesced 4-byte read and an LDS minimum, and D(r) is read and written
// once.  64 neighbours' records load side by side, and their entries are
// walked as one concatenated range, so short entry lists fill the wave.
// Bound by the gathered entries' loads (0.19 ms per round).  Weighted R-MAT-16:
// the pushes of a build took 22.6 ms; 10 gathered rounds take 1.9 and the
// pushes left 1.7.
constexpr uint32_t kPullWUnroll = 4;

__device__ inline void phase_pull_w(const BuildArgs& A, const Exec& X, uint32_t ib, uint32_t bs, const uint2* items,
                                    const uint32_t* nitems, uint32_t p, uint32_t rstamp, uint32_t bstamp,
                                    uint32_t* s_min, uint32_t* s_end) {
    const uint32_t lane = lane_id();
    const uint32_t W = A.W;
    if (X.zero_i < X.nq) X.qs[X.zero_i].hq[p ^ 1u] = 0;
    const uint32_t total = *nitems;
    for (uint32_t t = X.w; t < total; t += X.nw) {
        const uint2 it = items[t];
        const uint32_t r = it.x;
        if (r <= ib) continue;
        const uint32_t rel = min(r - ib, bs);  // roots ranked above r
        const uint64_t rbeg = A.rrow[r], rend = A.rrow[r + 1];
        const uint64_t beg = rbeg + (uint64_t)it.y * kPullSeg, end = min(rend, beg + kPullSeg);
        bool met = false;
        for (uint64_t e0 = beg; e0 < end; e0 += 64) {
            const uint64_t e = e0 + lane;
            bool act = e < end;
            const uint32_t c = act ? A.rcol[e] : 0u;
            const uint32_t wt = act ? A.rw[e] : 0u;
            const uint64_t at = act ? A.act_at[c] : 0ull;
            act = act && (uint32_t)(at >> 32) == rstamp - 1u;
            if (!ballot64(act)) continue;
            const uint2 rg = act ? A.act_rng[p][(uint32_t)at] : make_uint2(0u, 0u);
            uint64_t off = (act ? A.loff[c] : 0ull) + rg.x;
            const uint32_t pre = wave_excl_scan32(rg.y);
            const uint32_t tot = readlane32(pre + rg.y, 63);
            off -= pre;  // entry x of the concatenation is arena[off + x]
            wave_lds_sync();
            s_end[lane] = pre + rg.y;
            if (!met)
                for (uint32_t k = lane; k < 64u * W; k += 64) s_min[k] = ~0u;
            met = true;
            wave_lds_sync();
            for (uint32_t x0 = 0; x0 < tot; x0 += 64u * kPullWUnroll) {
                uint32_t ent[kPullWUnroll], w[kPullWUnroll];
#pragma unroll
                for (uint32_t u = 0; u < kPullWUnroll; ++u) {
                    const uint32_t x = x0 + 64u * u + lane;
                    // the neighbour whose entries hold x: the first whose end is above x
                    uint32_t l = 0;
#pragma unroll
                    for (uint32_t step = 32; step; step >>= 1)
                        if (s_end[l + step - 1u] <= x) l += step;
                    l = min(l, 63u);
                    const uint64_t o = shfl64(off, l);
                    w[u] = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(l * 4u), (int)wt);
                    ent[u] = x < tot ? A.arena[o + x] : ~0u;
                }
#pragma unroll
                for (uint32_t u = 0; u < kPullWUnroll; ++u) {
                    const uint32_t k = (ent[u] >> 8) - ib;
                    if (x0 + 64u * u + lane < tot && k < rel) atomicMin(&s_min[k], (ent[u] & 255u) + w[u]);
                }
            }
        }
        if (!met) continue;
        wave_lds_sync();
        // rows of one segment are this wave's alone; the segments of a longer
        // one meet in D(r) and msgs(r)
        const bool alone = rend - rbeg <= kPullSeg;
        bool any = false, over = false;
        for (uint32_t k0 = 0; k0 < rel; k0 += 64) {
            const uint32_t k = k0 + lane;
            const uint32_t m = k < rel ? s_min[k] : ~0u;
            bool low = false;
            if (m != ~0u) {
                uint8_t* pd = A.D + (size_t)r * A.bstride + k;
                const uint32_t old = *pd;
                // too long for the labels, and nothing shorter has come
                over = over || (m >= PLL_INF8 && old == PLL_INF8);
                low = m < PLL_INF8 && m < old;
                if (low && alone) *pd = (uint8_t)m;
                if (low && !alone) low = byte_atomic_min(pd, m);
            }
            const uint64_t bits = ballot64(low);
            if (!bits) continue;
            any = true;
            if (lane == 0)
                atomicOr((unsigned long long*)&A.msgs[(size_t)r * W + (k0 >> 6)], (unsigned long long)bits);
        }
        if (ballot64(over) && lane == 0) atomicOr(&A.ctr->error, PLL_ERR_DIST);
        enqueue_receivers(A, X, A.recv, p, rstamp, bstamp, r, any && lane == 0);
    }
}

// Gather phase for weighted graphs: the candidates of receiver v are the
// bits of msgs(v); candidate u_k has distance D(v)[k], staged in this
// wave's LDS s_thr (64 * W bytes).  Survivors are appended with that
// distance (a hub may already hold a longer entry from an earlier round;
// the batch end keeps the last one); the slot records where they start.
template <int WM>
__device__ inline void phase_check_w(const BuildArgs& A, const Exec& X, uint32_t ib, uint32_t bs, uint32_t p,
                                     uint32_t rstamp, uint4* s_thr, PhaseStats& st) {
    const uint32_t lane = lane_id();
    const uint32_t W = A.W;
    const uint32_t q = p ^ 1u;
    uint32_t pre;
    const uint32_t nrecv = shard_prefix(lane < X.nq ? X.qs[lane].recv[p] : 0u, pre);
    if (X.zero_i < X.nq) X.qs[X.zero_i].recv[q] = 0;
    const uint8_t* thr_bytes = reinterpret_cast<const uint8_t*>(s_thr);
    for (uint32_t i = X.w; i < nrecv; i += X.nw) {
        const uint32_t s = shard_of(X.nq, pre, i);
        const uint32_t v = A.recv[(size_t)s * X.seg + (i - readlane32(pre, s))];
        uint64_t mine = 0;
        if (lane < W) {
            const size_t at = (size_t)v * W + lane;
            mine = A.msgs[at];
            A.msgs[at] = 0;
        }
        const uint4* drow = reinterpret_cast<const uint4*>(A.D + (size_t)v * A.bstride);
        for (uint32_t c = lane; c < 4 * W; c += 64) s_thr[c] = drow[c];
        wave_lds_sync();
        const uint32_t len = A.llen[v];
        uint64_t off = A.loff[v];
        const uint64_t pw = prune_scan_w<WM>(A, off, len, mine, s_thr, ib, st);
        const uint64_t acc = lane < W ? (mine & ~pw) : 0ull;
        const uint32_t cnt = (uint32_t)__builtin_popcountll(acc);
        const uint32_t pos = wave_excl_scan32(cnt);
        const uint32_t total = readlane32(pos + cnt, 63);
        st.cand += __builtin_popcountll(mine);
        st.cost_pos += (unsigned long long)len * (uint32_t)__builtin_popcountll(acc);
        st.cost_neg += (unsigned long long)len * (uint32_t)__builtin_popcountll(mine & ~acc);
        if (lane == 0) {
            A.act_v[q][i] = v;
            A.act_rng[q][i] = make_uint2(len, total);
        }
        if (total != 0) {
            off = wave_reserve(A, X, v, off, len, A.lcap[v], total);
            if (off != ~0ull) {
                if (lane == 0) st.acc += total;
                const bool in_batch = v - ib < bs;
                const uint64_t lt = lanemask_lt();
                uint64_t todo = ballot64(acc != 0);
                while (todo) {
                    const uint32_t w = (uint32_t)__builtin_ctzll(todo);
                    todo &= todo - 1;
                    const uint64_t aw = readlane64(acc, w);
                    const uint32_t pwos = readlane32(pos, w);
                    if ((aw >> lane) & 1ull) {
                        const uint32_t k = w * 64u + lane;
                        const uint32_t dk = thr_bytes[k];
                        A.arena[off + len + pwos + __builtin_popcountll(aw & lt)] = pll_pack(ib + k, dk);
                        if (in_batch) {
                            A.T[(size_t)(ib + k) * A.bstride + (v - ib)] = (uint8_t)dk;
                            atomicOr((unsigned long long*)&A.rowmask[ib + k], 1ull << ((v - ib) >> 4));
                        }
                    }
                }
                if (lane == 0) {
                    A.llen[v] = len + total;
                    // for a pulled next round: where v's entries are, and its edges
                    A.act_at[v] = ((uint64_t)rstamp << 32) | i;
                    st.pulled += A.rrow[v + 1] - A.rrow[v];
                }
                enqueue_heavy(A, X, q, i, A.rrow[v + 1] - A.rrow[v]);
            } else if (lane == 0) {
                A.act_rng[q][i] = make_uint2(len, 0u);
            }
        }
        wave_lds_sync();
    }
}

// The byte table from the labels the batch's roots hold now (one wave per
// root): a build whose rounds outgrow the bit planes goes on with it.
__device__ inline void phase_table_fill(const BuildArgs& A, const Exec& X, uint32_t ib, uint32_t bs) {
    const uint32_t lane = lane_id();
    for (uint32_t k = X.w; k < bs; k += X.nw) {
        const uint32_t len = A.llen[ib + k];
        const uint64_t off = A.loff[ib + k];
        for (uint32_t i = lane; i < len; i += 64) {
            const uint32_t e = A.arena[off + i];
            const uint32_t h = e >> 8;
            A.T[(size_t)h * A.bstride + k] = (uint8_t)(e & 255u);
            if (h >= A.hot) atomicOr((unsigned long long*)&A.rowmask[h], 1ull << (k >> 4));
        }
    }
}

// Reset the distance table rows (or plane words) written during the batch.
// With HOT, planes 1 and 2 of the rows below kInitHot are zeroed whole (they
// hold bits of most roots, which would each zero the same words again).
// Bound by the scattered stores: R-MAT-20, all batches, 6.0 ms on the byte
// table, 4.2 so.
template <bool PLANES = false, bool HOT = false>
__device__ inline void phase_clear_table(const BuildArgs& A, const Exec& X, uint32_t ib, uint32_t bs) {
    const uint32_t lane = lane_id();
    if (HOT) {
        const uint32_t words = min(ib + bs, kInitHot) * A.W;  // 16-byte units of planes 1 and 2
        for (uint32_t i = X.w * 64u + lane; i < words; i += X.nw * 64u) {
            ulonglong2* row = reinterpret_cast<ulonglong2*>(A.P + (size_t)(i / A.W) * (PLL_PLANES * A.W));
            row[i % A.W] = make_ulonglong2(0ull, 0ull);
        }
    }
    // four waves per root: task t clears the 64-entry chunks c, c + 4, ...
    // of root k (t = 4k + c)
    for (uint32_t t = X.w; t < 4u * bs; t += X.nw) {
        const uint32_t k = t >> 2, c = t & 3u;
        const uint32_t u = ib + k;
        const uint32_t len = A.llen[u];
        const uint64_t off = A.loff[u];
        for (uint32_t i = 64u * c + lane; i < len; i += 256u) {
            const uint32_t e = A.arena[off + i];
            const uint32_t h = e >> 8;
            if (PLANES) {
                const uint32_t d = e & 255u;
                uint64_t* row = A.P + (size_t)h * (PLL_PLANES * A.W) + (k >> 6);
                if (HOT && d <= 2 && h < kInitHot) continue;
                if (d == 1) row[0] = 0;
                if (d != 0 && d <= PLL_PLANES) row[(max(d, 2u) - 1u) * A.W] = 0;
            } else {
                A.T[(size_t)h * A.bstride + k] = (uint8_t)PLL_INF8;
                if (h >= A.hot) A.rowmask[h] = 0;
            }
        }
        if (!PLANES && c == 0 && lane == 0 && u >= A.hot) A.rowmask[u] = 0;
    }
}

}  // namespace pll
