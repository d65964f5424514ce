// pa_api.cpp -- host side of the C ABI declared in include/pa.h.
//
// Validates the graph (paper section 1: undirected graph, binary weights),
// builds the device-friendly CSR, the dependency-level schedule of the sweep
// order, and the fixed-point tables of the Metropolis thresholds and
// resampling weights (FP64 exp on the host, then floor(2^32 * value)), lays
// out the caller's workspace and enqueues the step loop on the caller's
// stream. Device work is in pa_kernels.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <map>
#include <thread>
#include <new>
#include <vector>

#include "pa.h"
#include "pa_device.h"
#include "pa_host.h"

namespace pa_host {

thread_local char g_error[512] = "";

pa_status fail(pa_status st, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_error, sizeof g_error, fmt, ap);
    va_end(ap);
    return st;
}

pa_status hip_fail(hipError_t e, const char *what)
{
    return fail(PA_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

}  // namespace pa_host

using namespace pa_host;

extern "C" const char *pa_last_error(void) { return g_error; }

// --------------------------------------------------------------- create ----

extern "C" pa_status pa_create(pa_solver **out, int32_t n, const int32_t *row_ptr,
                               const int32_t *col, const int8_t *w)
{
    g_error[0] = 0;
    if (!out || !row_ptr || (!col && row_ptr && n > 0 && row_ptr[n] > 0) || (!w && col))
        return fail(PA_EINVAL, "pa_create: null pointer argument");
    *out = nullptr;
    if (n < 2 || n > kMaxN) return fail(PA_ERANGE, "pa_create: n=%d outside [2, %d]", n, kMaxN);
    if (row_ptr[0] != 0) return fail(PA_EINVAL, "pa_create: row_ptr[0] must be 0");
    for (int i = 0; i < n; ++i)
        if (row_ptr[i + 1] < row_ptr[i]) return fail(PA_EINVAL, "pa_create: row_ptr decreases at %d", i);
    const long long nnz = row_ptr[n];
    std::vector<std::vector<std::pair<int, int>>> rows(n);
    int dmax = 0;
    for (int i = 0; i < n; ++i) {
        const int d = row_ptr[i + 1] - row_ptr[i];
        if (d > kMaxDegree) return fail(PA_ERANGE, "pa_create: degree %d of node %d > %d", d, i, kMaxDegree);
        dmax = std::max(dmax, d);
        rows[i].reserve(d);
        for (int e = row_ptr[i]; e < row_ptr[i + 1]; ++e) {
            const int j = col[e];
            if (j < 0 || j >= n) return fail(PA_EINVAL, "pa_create: column %d out of range in row %d", j, i);
            if (j == i) return fail(PA_EINVAL, "pa_create: self loop at node %d", i);
            if (w[e] != 1 && w[e] != -1)
                return fail(PA_EINVAL, "pa_create: weight %d of edge (%d,%d) is not +-1", (int)w[e], i, j);
            rows[i].push_back({j, (int)w[e]});
        }
        std::sort(rows[i].begin(), rows[i].end());
        for (size_t q = 1; q < rows[i].size(); ++q)
            if (rows[i][q].first == rows[i][q - 1].first)
                return fail(PA_EINVAL, "pa_create: repeated neighbour %d in row %d", rows[i][q].first, i);
    }
    long long wsum = 0;
    for (int i = 0; i < n; ++i)
        for (auto &jw : rows[i]) {
            auto &rj = rows[jw.first];
            auto it = std::lower_bound(rj.begin(), rj.end(), std::make_pair(i, -2));
            if (it == rj.end() || it->first != i || it->second != jw.second)
                return fail(PA_EINVAL, "pa_create: edge (%d,%d) has no symmetric partner", i, jw.first);
            wsum += jw.second;
        }
    pa_solver *s = new (std::nothrow) pa_solver;
    if (!s) return fail(PA_ERANGE, "pa_create: out of host memory");
    s->n = n;
    s->nnz = nnz;
    s->dmax = dmax;
    s->w_tot = wsum / 2;
    s->row_ptr.resize(n + 1);
    s->col.resize(nnz);
    s->npos.resize(n);
    long long e = 0;
    for (int i = 0; i < n; ++i) {
        s->row_ptr[i] = (int)e;
        int np = 0;
        for (auto &jw : rows[i])
            if (jw.second > 0) { s->col[e++] = jw.first; ++np; }
        for (auto &jw : rows[i])
            if (jw.second < 0) { s->col[e++] = jw.first; s->has_neg = 1; }
        s->npos[i] = np;
    }
    s->row_ptr[n] = (int)e;
    s->edges.reserve(nnz / 2);
    for (int i = 0; i < n; ++i)
        for (auto &jw : rows[i])
            if (jw.first > i)
                s->edges.push_back((uint32_t)i | ((uint32_t)jw.first << 15) | (jw.second < 0 ? 1u << 30 : 0u));
    {
        // Fixed pseudo-random order (xorshift64 Fisher-Yates): concurrent
        // unions in the cluster move then rarely meet the same root.
        uint64_t z = 0x9E3779B97F4A7C15ull;
        for (size_t q = s->edges.size(); q > 1; --q) {
            z ^= z << 13;
            z ^= z >> 7;
            z ^= z << 17;
            std::swap(s->edges[q - 1], s->edges[z % q]);
        }
    }
    *out = s;
    return PA_OK;
}

extern "C" pa_status pa_destroy(pa_solver *s)
{
    if (!s) return PA_OK;
    if (s->has_run && s->stream) (void)hipStreamSynchronize(s->stream);
    if (s->stage_pending) (void)hipEventSynchronize(s->stage_ev);
    if (s->stage_ev) (void)hipEventDestroy(s->stage_ev);
    if (s->stage) (void)hipHostFree(s->stage);
    for (hipEvent_t e : s->ev) (void)hipEventDestroy(e);
    delete s;
    return PA_OK;
}

extern "C" pa_status pa_graph_info(const pa_solver *s, int64_t out[4])
{
    if (!s || !out) return fail(PA_EINVAL, "pa_graph_info: null argument");
    out[0] = s->n;
    out[1] = s->nnz;
    out[2] = s->w_tot;
    out[3] = s->dmax;
    return PA_OK;
}

// ----------------------------------------------------------------- plan ----

// Adaptive steps reweight a jump of j grid points by beta[j] - beta[0], which
// is the jump's own increase beta[g + j] - beta[g] only on an evenly spaced
// grid. Returns the index of the first spacing beta[k + 1] - beta[k] that
// differs from the mean spacing by more than 1e-9 of it plus 8 ulps of the
// largest |beta| (the rounding of a linear grid in FP64), or -1 if none does.
static int uneven_grid(const double *beta, int K)
{
    if (K < 3) return -1;
    const double h = (beta[K - 1] - beta[0]) / (double)(K - 1);
    const double big = std::max(std::fabs(beta[0]), std::fabs(beta[K - 1]));
    const double tol = 1e-9 * std::fabs(h) + 8.0 * std::ldexp(big, -52);
    for (int k = 0; k + 1 < K; ++k)
        if (std::fabs((beta[k + 1] - beta[k]) - h) > tol) return k;
    return -1;
}

pa_status pa_host::check_schedule(const pa_solver *s, const pa_schedule *sch, int R)
{
    if (!s || !sch) return fail(PA_EINVAL, "null solver or schedule");
    if (sch->n_steps < 1) return fail(PA_EINVAL, "n_steps must be >= 1");
    if (!sch->beta) return fail(PA_EINVAL, "beta is null");
    if (sch->sweeps_per_step < 1 || sch->sweeps_per_step > 65535)
        return fail(PA_ERANGE, "sweeps_per_step=%d outside [1, 65535]", sch->sweeps_per_step);
    for (int k = 0; k < sch->n_steps; ++k) {
        const double b = sch->beta[k];
        if (!std::isfinite(b) || b < 0.0) return fail(PA_EINVAL, "beta[%d] is not finite and >= 0", k);
        if (k > 0 && b < sch->beta[k - 1]) return fail(PA_EINVAL, "beta decreases at step %d", k);
    }
    if (sch->as_enable != 0 && sch->as_enable != 1) return fail(PA_EINVAL, "as_enable must be 0 or 1");
    if (sch->as_enable) {
        if (sch->as_stall_steps < 1) return fail(PA_EINVAL, "as_stall_steps must be >= 1");
        if (sch->as_max_level < 0 || sch->as_max_level > 15)
            return fail(PA_ERANGE, "as_max_level outside [0, 15]");
        if (sch->as_frozen_inv < 1) return fail(PA_EINVAL, "as_frozen_inv must be >= 1");
        if (!(sch->as_gamma > 0.0 && sch->as_gamma <= 1.0)) return fail(PA_EINVAL, "as_gamma outside (0, 1]");
    }
    if (sch->nl_period < 0) return fail(PA_EINVAL, "nl_period must be >= 0");
    if (sch->field_bits != 0 && sch->field_bits != 8 && sch->field_bits != 16)
        return fail(PA_EINVAL, "field_bits=%d is not 0, 8 or 16", sch->field_bits);
    if (sch->field_bits == 8 && s->dmax > 127)
        return fail(PA_ERANGE, "a local field reaches the maximum degree %d, beyond 8-bit fields", s->dmax);
    if (R < 1 || R > kMaxR) return fail(PA_ERANGE, "R=%d outside [1, %d]", R, kMaxR);
    if (sch->nl_kind != 0 && sch->nl_kind != 1) return fail(PA_EINVAL, "nl_kind must be 0 or 1");
    if (sch->beta_adapt != 0 && sch->beta_adapt != 1) return fail(PA_EINVAL, "beta_adapt must be 0 or 1");
    if (sch->beta_adapt) {
        if (sch->adapt_jump < 1 || sch->adapt_jump > pa::kMaxJump)
            return fail(PA_EINVAL, "adapt_jump must be in [1, %d]", pa::kMaxJump);
        if (sch->adapt_den < 1 || sch->adapt_den > 65536 || sch->adapt_num < 0 || sch->adapt_num > sch->adapt_den)
            return fail(PA_EINVAL, "adaptive target needs 0 <= adapt_num <= adapt_den <= 65536, den >= 1");
        const int bad = uneven_grid(sch->beta, sch->n_steps);
        if (bad >= 0)
            return fail(PA_EINVAL, "adaptive steps need an evenly spaced beta grid (spacing %d differs)", bad);
    }
    if (sch->nl_period > 0 && sch->nl_kind == 0 && (R & 1))
        return fail(PA_EINVAL, "pair cluster moves pair replicas: R must be even");
    if (sch->tile_replicas != 0 && sch->tile_replicas != 4 && sch->tile_replicas != 8 &&
        sch->tile_replicas != 16 && sch->tile_replicas != 32 && sch->tile_replicas != 64)
        return fail(PA_EINVAL, "tile_replicas must be 0, 4, 8, 16, 32 or 64");
    if (sch->record < 0 || sch->record > 3) return fail(PA_EINVAL, "record must be in [0, 3]");
    if (sch->wg_threads != 0 && (sch->wg_threads < 64 || sch->wg_threads > 1024 || sch->wg_threads % 64))
        return fail(PA_EINVAL, "wg_threads must be 0 or a multiple of 64 in [64, 1024]");
    if (sch->order) {
        std::vector<char> seen(s->n, 0);
        for (int t = 0; t < s->n; ++t) {
            const int i = sch->order[t];
            if (i < 0 || i >= s->n || seen[i]) return fail(PA_EINVAL, "order is not a permutation (position %d)", t);
            seen[i] = 1;
        }
    }
    return PA_OK;
}

// Dependency levels of the sweep order: level(i) = 1 + max level of the
// neighbours visited before i (0 if none). Nodes of one level are pairwise
// non-adjacent, and visiting levels in increasing order reproduces the
// sequential sweep exactly, since each attempt only reads its neighbours.
void pa_host::build_levels(const pa_solver *s, const int32_t *order, Levels &p)
{
    const int n = s->n;
    const int *row_ptr = s->row_ptr.data(), *col = s->col.data();
    std::vector<int> lvl(n, -1);                // -1: not visited yet
    std::vector<int> by_degree(s->dmax + 2, 0);
    int nl = 0;
    for (int t = 0; t < n; ++t) {
        const int i = order ? order[t] : t;
        int l = -1, l1 = -1, l2 = -1, l3 = -1;  // (four maxima: long rows wait for no chain)
        int e = row_ptr[i];
        for (; e + 4 <= row_ptr[i + 1]; e += 4) {
            l = std::max(l, lvl[col[e]]);
            l1 = std::max(l1, lvl[col[e + 1]]);
            l2 = std::max(l2, lvl[col[e + 2]]);
            l3 = std::max(l3, lvl[col[e + 3]]);
        }
        for (; e < row_ptr[i + 1]; ++e) l = std::max(l, lvl[col[e]]);
        l = std::max(std::max(l, l1), std::max(l2, l3)) + 1;
        lvl[i] = l;
        nl = std::max(nl, l + 1);
        ++by_degree[s->dmax - (row_ptr[i + 1] - row_ptr[i]) + 1];
    }
    p.n_levels = nl;
    p.level_off.assign(nl + 1, 0);
    for (int i = 0; i < n; ++i) p.level_off[lvl[i] + 1]++;
    for (int l = 0; l < nl; ++l) p.level_off[l + 1] += p.level_off[l];
    // Within a level the visiting order is free; grouping equal degrees
    // keeps the slots of one pass (which loop to their largest degree) even.
    // The nodes by falling degree first (visiting order among equals), then
    // dealt to their levels in that order.
    for (int d = 0; d < s->dmax; ++d) by_degree[d + 1] += by_degree[d];
    std::vector<int> nodes(n);
    for (int t = 0; t < n; ++t) {
        const int i = order ? order[t] : t;
        nodes[by_degree[s->dmax - (row_ptr[i + 1] - row_ptr[i])]++] = i;
    }
    std::vector<int> fill(p.level_off.begin(), p.level_off.end() - 1);
    p.sched.assign(n, 0);
    for (int i : nodes) p.sched[fill[lvl[i]]++] = i;
}

// Adjacency blocks in schedule order, one fixed-size block per slot:
// u32 {LDS byte offset of the node's spin word, degree, node, 0}, then the LDS
// byte offsets of the neighbours' words, padded with the zero word to a
// multiple of 4 entries. A neighbour joined by a negative weight points at
// the complemented copy of its spin word (word n + j), so every entry counts
// "w_ij x_j = +1" by a plain bit read. Each wave's pass stream lists
// {first slot, largest degree among the pass's slots}.
// direct: 1 or 0 imposes the entry form of kernel 1's blocks, -1 takes
// offsets whenever they fit 16 bits.
static void build_blocks(const pa_solver *s, Plan &p, int direct)
{
    const int n = s->n;
    if (p.kind == 1) {
        // Kernel 1: u16 {node, degree, neighbour record indices...}, padded
        // with the zero record's index to 8m - 2 entries (a multiple of 16
        // bytes with the header, at least the degree rounded up to 4).
        // Negative edges name the complemented record n + j (record mode 1)
        // or carry a sign bit, bit 0 of a byte offset or bit 15 of an index
        // (record mode 2). Record indices
        // count from the start of LDS (the threshold table occupies the first
        // rb records). Blocks n .. n + threads - 1 are all-padding blocks:
        // a lane reads the block of slot (first slot of its round + lane),
        // which may lie past the last node.
        const int rb = pa::kBytesRecBase / p.W;     // records start after the threshold table
        const int zrec = p.bsg == 1 ? 2 * n : n;    // index of the zero record
        // Entries are LDS byte offsets when every record's offset fits in 16
        // bits (one instruction to decode), else record indices.
        p.direct = direct >= 0 ? direct : pa::kBytesRecBase + zrec * p.W <= 0xFFFF;
        auto enc = [&](int rec) {
            return (uint16_t)(p.direct ? pa::kBytesRecBase + rec * p.W : rec + rb);
        };
        const uint16_t zi = enc(zrec);
        const int need = 4 * ((std::max(s->dmax, 1) + 3) / 4);
        int capk = 6;
        while (capk < need) capk += 8;
        p.block_bytes = 2 * (2 + capk);
        const int bw16 = p.block_bytes / 2;
        std::vector<uint16_t> b16((size_t)(n + p.threads) * bw16 + 32, zi);
        for (int t = 0; t < n; ++t) {
            const int i = p.sched[t];
            uint16_t *b = &b16[(size_t)t * bw16];
            const int e0 = s->row_ptr[i], e1 = s->row_ptr[i + 1];
            b[0] = (uint16_t)i;
            b[1] = (uint16_t)(e1 - e0);
            for (int e = e0; e < e1; ++e) {
                const int j = s->col[e];
                const bool neg = e >= e0 + s->npos[i];
                if (p.bsg == 2)
                    b[2 + (e - e0)] = (uint16_t)(enc(j) | (neg ? (p.direct ? 1u : 0x8000u) : 0u));
                else
                    b[2 + (e - e0)] = enc(neg ? n + j : j);
            }
        }
        for (int t = n; t < n + p.threads; ++t) {
            b16[(size_t)t * bw16] = 0;
            b16[(size_t)t * bw16 + 1] = 0;
        }
        p.blocks.assign((b16.size() + 1) / 2, 0u);
        std::memcpy(p.blocks.data(), b16.data(), b16.size() * sizeof(uint16_t));
        // Rounds: a level is cut into chunks of one node per thread.
        p.rounds.clear();
        for (int l = 0; l < p.n_levels; ++l) {
            const int beg = p.level_off[l], end = p.level_off[l + 1];
            for (int f = beg; f < end; f += p.threads) {
                p.rounds.push_back(f);
                p.rounds.push_back(end);
                p.rounds.push_back(f + p.threads >= end ? 1 : 0);
                p.rounds.push_back(0);
            }
        }
        p.n_rounds = (int)p.rounds.size() / 4;
        // A byte accumulator gains at most d_max per round; the kernel runs
        // rounds in pairs, so the count is even (d_max <= 127 keeps it >= 2).
        p.flush_every = std::max(2, (255 / std::max(s->dmax, 1)) & ~1);
        return;
    }
    const int cap = 4 * ((std::max(s->dmax, 1) + 3) / 4);
    p.block_bytes = 16 + 4 * cap;
    const int bw = p.block_bytes / 4;
    const int NS = 64 / p.W, NW = p.threads / 64;
    const int sh = p.W == 16 ? 1 : (p.W == 32 ? 2 : 3);
    const uint32_t zero = (uint32_t)(p.sgn ? 2 * n : n) << sh;
    p.blocks.assign((size_t)n * bw + 32, zero);
    for (int t = 0; t < n; ++t) {
        const int i = p.sched[t];
        uint32_t *b = &p.blocks[(size_t)t * bw];
        const int e0 = s->row_ptr[i], e1 = s->row_ptr[i + 1];
        b[0] = (uint32_t)i << sh;
        b[1] = (uint32_t)(e1 - e0);
        b[2] = (uint32_t)i;
        b[3] = 0;
        for (int e = e0; e < e1; ++e) {
            const int j = s->col[e];
            const bool neg = e >= e0 + s->npos[i];
            b[4 + (e - e0)] = (uint32_t)(neg ? n + j : j) << sh;
        }
    }
    std::vector<std::vector<int>> st(NW);
    for (int l = 0; l < p.n_levels; ++l) {
        const int beg = p.level_off[l], end = p.level_off[l + 1], Lsz = end - beg;
        for (int w = 0; w < NW; ++w) {
            const int npass = Lsz > w * NS ? (Lsz - w * NS + NW * NS - 1) / (NW * NS) : 0;
            for (int q = 0; q < npass; ++q) {
                const int base = beg + w * NS + q * NW * NS;
                int md = 0;
                for (int t = base; t < base + NS && t < end; ++t) {
                    const int i = p.sched[t];
                    md = std::max(md, s->row_ptr[i + 1] - s->row_ptr[i]);
                }
                st[w].push_back(base);
                st[w].push_back(md);
            }
        }
    }
    size_t qmax = 0;
    for (auto &v : st) qmax = std::max(qmax, v.size() / 2);
    p.qpad = (int)qmax + 4;
    p.stream.assign((size_t)NW * p.qpad * 2, 0);
    for (int w = 0; w < NW; ++w)
        for (int q = 0; q < p.qpad; ++q) {
            const bool have = (size_t)q < st[w].size() / 2;
            p.stream[((size_t)w * p.qpad + q) * 2] = have ? st[w][2 * q] : -1;
            p.stream[((size_t)w * p.qpad + q) * 2 + 1] = have ? st[w][2 * q + 1] : 0;
        }
}

// Parts of at most `most` that `count` >= 1 is cut into. (One, in most levels:
// no division then.)
static inline int parts(int count, int most)
{
    return count <= most ? 1 : (count + most - 1) / most;
}

bool pa_host::fuse_draws(const pa_solver *s, int n_levels)
{
    return (s->dmax == 4 || s->dmax == 2) && s->nnz == (long long)s->n * s->dmax && s->n + 256 <= 0x7FFF &&
           s->n >= 256 * n_levels;
}

// Nodes of a level that a wave of the tile form takes together.
struct Item {
    int slot, count, lp, rows, per;     // per: entries a lane, of the largest node
    int lanes() const { return count << lp; }
};

// The levels cut into items. Entries a lane's block holds: 6 + 8 after a short
// header, 4 in the first row after a long one, 8 more with 16-bit counters (16
// in all with sign bits), four with draws in registers. A node of a larger
// degree takes 2^lp lanes. An item that leaves half its lanes free spreads its
// nodes over more of them down to one row a lane: the chain of a level shortens
// with the entries read in turn.
static void cut_levels(const pa_solver *s, const Levels &v, bool long_head, bool d16, int fuse,
                       std::vector<Item> &cut, int *level_item)
{
    const int e0 = long_head ? 4 : 6;
    const int most = fuse ? e0 : !d16 ? e0 + 8 : long_head ? 16 : e0 + 16, lp_max = d16 ? 6 : 4;
    cut.reserve(v.n_levels + s->n / 32);
    for (int l = 0; l < v.n_levels; ++l) {
        for (int t = v.level_off[l]; t < v.level_off[l + 1];) {
            const int i = v.sched[t], md = s->row_ptr[i + 1] - s->row_ptr[i];
            auto per_lane = [&](int lp) { return (md + (1 << lp) - 1) >> lp; };
            Item it{t, 0, 0, 1, 0};
            while (per_lane(it.lp) > most) ++it.lp;
            it.count = std::min(v.level_off[l + 1] - t, 64 >> it.lp);
            while (it.lp < lp_max && per_lane(it.lp) > e0 && it.count << (it.lp + 1) <= 64) ++it.lp;
            it.per = per_lane(it.lp);
            it.rows = it.per <= e0 ? 1 : 1 + (it.per - e0 + 7) / 8;
            cut.push_back(it);
            t += it.count;
        }
        if (level_item) level_item[l + 1] = (int)cut.size();
    }
}

long long pa_host::tile_rows(const pa_solver *s, const Levels &v, bool long_head)
{
    std::vector<Item> cut;
    cut_levels(s, v, long_head, s->dmax > kMaxBytesDegree, 0, cut, nullptr);
    long long rows = 0;
    for (const Item &it : cut) rows += it.rows;
    return rows;
}

// The tile form's item streams and blocks (their layout is described at
// sweep_tile_kernel). Every level is cut into items of at most 64 lanes, dealt over the
// waves; levels are gathered into chunks whose draws fit half the draw buffer,
// and the draws of a chunk are dealt, as items of 64 slots, into the places
// that the chunk before it leaves free. Without `fill` only the sizes are set:
// they follow from the cut and from where the draws go, and no row is written.
static void build_tile_plan(const pa_solver *s, Plan &p, bool fill)
{
    const int n = s->n, W = p.W, nw = p.threads / 64;
    const bool d16 = p.deg == 2;
    const bool long_head = p.bsg != 0;
    const int e0 = long_head ? 4 : 6;
    std::vector<Item> cut;
    std::vector<int> level_item(p.n_levels + 1, 0);
    cut_levels(s, p, long_head, d16, p.fuse, cut, level_item.data());
    p.n_rounds = 0;
    for (int l = 0; l < p.n_levels; ++l) p.n_rounds += parts(level_item[l + 1] - level_item[l], nw);

    // Chunks: runs of items whose slots fit a half of the draw buffer.
    const int cap = pa::tile_draw_slots(W, d16) / 128 * 64;
    p.draw_half = cap * (d16 ? 2 * W : W);
    std::vector<int> chunk_item{0};             // first item of each chunk, then the end
    for (int c = 0, slot = 0; c < (int)cut.size(); ++c)
        if (!p.fuse && cut[c].slot + cut[c].count - slot > cap) {
            chunk_item.push_back(c);
            slot = cut[c].slot;
        }
    chunk_item.push_back((int)cut.size());
    const int n_chunks = (int)chunk_item.size() - 1;
    auto chunk_slot = [&](int c) { return c < n_chunks ? cut[chunk_item[c]].slot : n; };

    // An item's wave: a level's items are dealt to the waves in turn; where
    // its item would stand alone (or nearly: at most a quarter more items than
    // levels) wave 0 takes the levels by itself and needs no barrier between.
    const bool solo = nw >= 2 && (long long)cut.size() * 4 <= 5LL * p.n_levels;
    std::vector<int> item_wave(cut.size(), 0);
    for (int l = 0, c = 1; l < p.n_levels && !solo; ++l)
        for (int q = level_item[l], k = 0; q < level_item[l + 1]; ++q) {
            if (q == chunk_item[c]) {           // a chunk's first item
                ++c;
                k = 0;
            }
            item_wave[q] = k;
            k = k + 1 < nw ? k + 1 : 0;
        }

    // Places of the blocks: the draw items' nodes, then the levels' rows.
    const int rec_words = 8;            // u16 per lane and row
    std::vector<int> draw_at(n_chunks, 0);      // uint4 offset of a chunk's draw blocks
    std::vector<int> draw_items(n_chunks, 0);
    size_t u4 = 0;
    if (!p.fuse)
        for (int c = 0; c < n_chunks; ++c) {
            draw_at[c] = (int)u4;
            draw_items[c] = (chunk_slot(c + 1) - chunk_slot(c) + 63) / 64;
            u4 += 64 * (size_t)draw_items[c];
        }
    std::vector<int> block_at(cut.size());
    for (size_t c = 0; c < cut.size(); ++c) {
        block_at[c] = (int)u4;
        u4 += (size_t)cut[c].rows * (cut[c].lanes() + 1);
    }
    u4 += 2 * 65;                               // rows that the last items do not have
    p.row_bytes = u4 * sizeof(uint16_t) * rec_words;

    // Streams. An interval runs from barrier to barrier: a level, or a run of
    // levels that wave 0 takes by itself. Its items are cut[q0 .. q1).
    struct Interval {
        int q0, q1;
        int longest;                            // items of its longest wave
        int wave;                               // where one more draw lengthens it least
        long long cost;                         //   and by how much (2^32: it does)
    };
    struct Draw {
        int iv, wave, t;
    };
    std::vector<std::vector<int2>> st(fill ? nw : 0);
    std::vector<int> st_len(nw, 0);
    std::vector<Interval> iv;
    std::vector<int> len;                       // items of each interval and wave
    std::vector<Draw> placed;
    const int2 nothing{0, pa::item_word(0, 0, 1, 0, 0)};
    for (int c = 0, l = 0; c < n_chunks; ++c) {
        iv.clear();
        int wave0_run = 0;                      // the open interval is wave 0's alone
        for (int q = chunk_item[c]; q < chunk_item[c + 1];) {
            while (level_item[l + 1] <= q) ++l;
            const int end = std::min(level_item[l + 1], chunk_item[c + 1]);
            const int alone = solo || level_item[l + 1] - level_item[l] == 1;
            if (iv.empty() || !(alone && wave0_run)) {
                iv.push_back(Interval{q, q, 0, 0, 0});
                wave0_run = alone;
            }
            iv.back().q1 = q = end;
        }
        len.assign(iv.size() * nw, 0);
        for (size_t v = 0; v < iv.size(); ++v)
            for (int q = iv[v].q0; q < iv[v].q1; ++q) ++len[v * nw + item_wave[q]];
        const int c2 = c + 1 < n_chunks ? c + 1 : 0;
        placed.clear();
        if (!p.fuse) {
            // The next chunk's draws, each where it lengthens its interval
            // least (wave 0 last).
            auto offer = [&](size_t v) {
                const int *m = &len[v * nw];
                iv[v].longest = *std::max_element(m, m + nw);
                iv[v].wave = -1;
                for (int w = nw - 1; w >= 0; --w) {
                    const long long more = (long long)m[w] + 1;
                    const long long cost = more > iv[v].longest ? (1LL << 32) + more : more - iv[v].longest;
                    if (iv[v].wave < 0 || cost < iv[v].cost) {
                        iv[v].wave = w;
                        iv[v].cost = cost;
                    }
                }
            };
            for (size_t v = 0; v < iv.size(); ++v) offer(v);
            for (int t = 0; t < draw_items[c2]; ++t) {
                size_t best = 0;
                for (size_t v = 1; v < iv.size(); ++v)
                    if (iv[v].cost < iv[best].cost) best = v;
                placed.push_back(Draw{(int)best, iv[best].wave, t});
                ++len[best * nw + iv[best].wave];
                offer(best);
            }
            std::stable_sort(placed.begin(), placed.end(), [](const Draw &x, const Draw &y) { return x.iv < y.iv; });
        }
        const int kind = c + 1 < n_chunks ? 2 : 3;
        for (size_t v = 0, d = 0; v < iv.size(); ++v) {
            const bool chunk_end = v + 1 == iv.size(), sweep_end = chunk_end && c + 1 == n_chunks;
            // (The sweep's last barrier is the kernel's own.)
            const int flags = (sweep_end ? 0 : pa::kItemBarrier) | (chunk_end && !p.fuse ? pa::kItemChunk : 0);
            for (int w = 0; w < nw; ++w) st_len[w] += flags != 0 && len[v * nw + w] == 0 ? 1 : len[v * nw + w];
            if (!fill) continue;
            for (int q = iv[v].q0; q < iv[v].q1; ++q) {
                const Item &it = cut[q];
                st[item_wave[q]].push_back(
                    int2{block_at[q] * 16,
                         pa::item_word(it.lanes(), p.fuse ? 0 : it.slot - chunk_slot(c), it.rows, it.lp, 1)});
            }
            for (; d < placed.size() && placed[d].iv == (int)v; ++d)
                st[placed[d].wave].push_back(
                    int2{(draw_at[c2] + 64 * placed[d].t) * 16, pa::item_word(63, 64 * placed[d].t, 1, 0, kind)});
            for (int w = 0; w < nw && flags != 0; ++w) {
                if (len[v * nw + w] == 0) st[w].push_back(nothing);
                st[w].back().y |= pa::item_word(0, 0, 1, 0, flags);
            }
        }
    }
    // Every stream has an even count of items, and its first three again.
    p.item_ints = 0;
    p.streams.assign((size_t)4 * nw, 0);
    for (int w = 0; w < nw; ++w) {
        const int even = st_len[w] + (st_len[w] & 1);
        int *head = &p.streams[(size_t)4 * w];
        head[0] = (int)p.item_ints / 2;
        head[1] = even;
        head[2] = draw_at[0];
        head[3] = draw_items[0];
        p.item_ints += 2 * ((size_t)even + 3);
    }
    if (!fill) return;
    p.items.clear();
    p.items.reserve(p.item_ints);
    for (std::vector<int2> &it : st) {
        if (it.size() & 1) it.push_back(nothing);
        const size_t m = it.size();
        for (size_t q = 0; q < m + 3; ++q) {
            const int2 v = m == 0 ? nothing : it[q % m];
            p.items.push_back(v.x);
            p.items.push_back(v.y);
        }
    }

    // The blocks' contents.
    const int rec0 = pa::tile_record(W, p.fuse, 0);     // record numbers follow one another
    const int *sched = p.sched.data(), *row_ptr = s->row_ptr.data(), *col = s->col.data();
    p.rows.assign(u4 * rec_words, 0);
    uint16_t *const rows = p.rows.data();
    for (int c = 0; c < (p.fuse ? 0 : n_chunks); ++c) {
        uint16_t *b = rows + (size_t)draw_at[c] * rec_words;
        for (int slot = chunk_slot(c); slot < chunk_slot(c + 1); ++slot, b += rec_words) b[0] = (uint16_t)sched[slot];
    }
    // A row is two words of four u16: a row of one record throughout, and the
    // first k of four entries followed by `pad`.
    auto all = [](int rec) { return 0x0001000100010001ull * (uint16_t)rec; };
    auto put = [](uint16_t *b, uint64_t v) { std::memcpy(b, &v, sizeof v); };
    auto four = [](const uint16_t *e, int k, uint64_t pad) {
        if (k <= 0) return pad;
        uint64_t v;
        std::memcpy(&v, e, sizeof v);
        const uint64_t past = k >= 4 ? 0 : ~0ull << 16 * k;
        return (v & ~past) | (pad & past);
    };
    std::vector<uint16_t> entry(s->dmax + 8);   // a node's entries
    const uint16_t neg_byte = W == 4 ? 0x01 : 0x11;
    for (size_t c = 0; c < cut.size(); ++c) {
        const Item &it = cut[c];
        const int lanes = it.lanes();
        const size_t stride = (size_t)(lanes + 1) * rec_words;
        uint16_t *const block = rows + (size_t)block_at[c] * rec_words;
        const int dummy = rec0 + (p.bsg == 1 ? 2 * n : n) + item_wave[c];
        uint16_t *spare = block + (size_t)lanes * rec_words;
        for (int r = 0; r < it.rows; ++r) {
            put(spare + r * stride, all(dummy));
            put(spare + r * stride + 4, all(dummy));
        }
        spare[1] = 0;
        // A FUSE block: {record, node}, a byte per neighbour where its edge is
        // negative, four neighbours. A dummy's first degree / 2 are.
        if (p.fuse) {
            spare[2] = (uint16_t)(s->dmax == 4 ? neg_byte * 0x0101 : neg_byte);
            spare[3] = 0;
            uint16_t *h = block;
            for (int lane = 0; lane < lanes; ++lane, h += rec_words) {
                const int i = sched[it.slot + lane];
                const int *nb = col + row_ptr[i];
                put(h, (uint16_t)(rec0 + i) | (uint64_t)i << 16);
                put(h + 4, all(rec0 + i));
                for (int q = 0; q < s->dmax; ++q) {
                    h[4 + q] = (uint16_t)(rec0 + nb[q]);
                    if (q >= s->npos[i]) h[2 + q / 2] = (uint16_t)(h[2 + q / 2] | neg_byte << 8 * (q % 2));
                }
            }
            continue;
        }
        if (long_head) spare[3] = p.bsg == 1 ? (uint16_t)dummy : 0;
        const int comp = p.bsg == 1 ? n : 0;
        uint16_t *h = block;
        for (int g = 0; g < it.count; ++g) {
            const int i = sched[it.slot + g], d = row_ptr[i + 1] - row_ptr[i], own = rec0 + i;
            const uint64_t pad = all(own);
            const int *nb = col + row_ptr[i];
            for (int t = 0; t < d; ++t) entry[t] = (uint16_t)(rec0 + nb[t]);
            for (int t = s->npos[i]; t < d && comp != 0; ++t) entry[t] = (uint16_t)(entry[t] + comp);
            for (int part = 0; part < 1 << it.lp; ++part, h += rec_words) {
                // Entries q0 .. q0 + m - 1 of the row, the first `pos` of them positive.
                const int q0 = std::min(d, part * it.per), m = std::min(d - q0, it.per);
                const uint16_t *e = entry.data() + q0;
                uint64_t head = (uint64_t)own | (uint64_t)d << 16;
                if (!long_head) {
                    // (The third and fourth u16 are entries 4 and 5.)
                    head |= (four(e + 4, std::min(m - 4, 2), pad) << 32);
                } else if (p.bsg == 1) {
                    head |= (uint64_t)(own + n) << 48;
                } else {
                    const int pos = std::min(std::max(s->npos[i] - q0, 0), m);
                    head |= (uint64_t)(((1u << m) - 1u) & ~((1u << pos) - 1u)) << 48;
                }
                put(h, head);
                put(h + 4, four(e, m, pad));
                uint16_t *b = h + stride;
                for (int r = 1, t = e0; r < it.rows; ++r, b += stride, t += 8) {
                    put(b, four(e + t, m - t, pad));
                    put(b + 4, four(e + t + 4, m - t - 4, pad));
                }
            }
        }
    }
}

// floor(2^32 * exp(-(beta * 2m))): the acceptance threshold of an uphill
// flip raising E by 2m at inverse temperature beta.
static uint64_t threshold_fixed(double beta, int m)
{
    const double x = std::exp(-(beta * (double)(2 * m)));
    return (uint64_t)std::floor(std::ldexp(x, 32));
}

// floor(2^32 (1 - exp(-2 beta))): activation of a satisfied unit bond in the
// single-replica cluster update (1 - exp as -expm1 in FP64).
static uint64_t bond_fixed(double beta)
{
    const double q = -std::expm1(-2.0 * beta);
    return (uint64_t)std::floor(std::ldexp(q, 32));
}

// floor(2^32 * exp(-(dbeta * n))): Boltzmann reweighting factor of a replica
// n above the population minimum when beta grows by dbeta.
static uint64_t weight_fixed(double dbeta, long long n)
{
    const double x = std::exp(-(dbeta * (double)n));
    return (uint64_t)std::floor(std::ldexp(x, 32));
}

// Calls fn(k0, k1) over [0, K) in contiguous chunks, on up to 8 host threads
// when the work (entries) is large enough to pay for them.
static void parallel_rows(int K, long long work, const std::function<void(int, int)> &fn)
{
    const unsigned hw = std::max(1u, std::thread::hardware_concurrency());
    const int nt = (int)std::min<long long>({8, (long long)hw, K, work / 20000 + 1});
    if (nt <= 1) {
        fn(0, K);
        return;
    }
    std::vector<std::thread> pool;
    const int per = (K + nt - 1) / nt;
    for (int t = 1; t < nt; ++t) {
        const int k0 = t * per, k1 = std::min(K, k0 + per);
        if (k0 < k1) pool.emplace_back(fn, k0, k1);
    }
    fn(0, std::min(K, per));
    for (auto &th : pool) th.join();
}

int Plan::sweep_lds(const pa_solver *s) const
{
    if (kind == 2) return pa::sweep_lds_bytes(W, sgn, s->n, s->dmax, threads);
    if (ahead) return pa::sweep_tile_lds(W, bsg == 1 ? 1 : 0, s->n, fuse);
    return pa::sweep_bytes_lds(W, bsg == 1 ? 1 : 0, s->n, s->dmax);
}

// Workspace bytes of the parts that depend on the sweep kernel's form: its
// plan, its threshold rows and what a workgroup leaves behind.
static size_t tail_bytes(const pa_solver *s, const Plan &p, size_t thr)
{
    return align_up(thr * (size_t)p.K * p.lmax1 * (s->dmax + 1)) + align_up(sizeof(uint64_t) * p.nblk) +
           align_up(sizeof(uint32_t) * (size_t)p.nblk * p.nw32);
}

static size_t general_bytes(const pa_solver *s, const Plan &p)
{
    const int n = s->n;
    size_t blocks, stream = 0;
    if (p.kind == 1) {
        const int need = 4 * ((std::max(s->dmax, 1) + 3) / 4);
        int capk = 6;
        while (capk < need) capk += 8;
        blocks = 4 * (((size_t)(n + p.threads) * (2 + capk) + 32 + 1) / 2);
        for (int l = 0; l < p.n_levels; ++l)
            stream += 16 * (size_t)parts(p.level_off[l + 1] - p.level_off[l], p.threads);
    } else {
        const int NS = 64 / p.W, NW = p.threads / 64;
        blocks = 4 * ((size_t)n * (4 + 4 * ((std::max(s->dmax, 1) + 3) / 4)) + 32);
        size_t passes = 0;
        for (int l = 0; l < p.n_levels; ++l)
            passes += (size_t)parts(p.level_off[l + 1] - p.level_off[l], NW * NS);
        stream = 8 * (size_t)NW * (passes + 4);
    }
    return align_up(sizeof(int) * n) + align_up(sizeof(int) * (p.n_levels + 1)) + align_up(blocks) +
           align_up(stream) + tail_bytes(s, p, sizeof(uint64_t));
}

static size_t tile_bytes(const pa_solver *s, const Plan &p)
{
    return align_up(p.row_bytes) + align_up(sizeof(int) * p.item_ints) + align_up(sizeof(int) * p.streams.size()) +
           tail_bytes(s, p, sizeof(uint32_t));
}

// A compute unit holds 24 to 32 waves of the tile kernel; a workgroup takes its
// share of them (us a launch of 10 sweeps, 5 on tori). One alone takes 1,024
// threads (n = 7,000, degree 4, R = 1,024: 143, with 512 160), on small levels
// 512 (n = 4,000, degree 12, 133 nodes a level: 146, with 1,024 164). Two, and
// more on levels of more than 160 nodes, take 512 each (n = 7,000, degree 12, R =
// 16,384: 1,160, with 256 1,400; R = 4,096: 346, with 768 369), four on smaller
// levels 256 (n = 4,000, degree 12, R = 16,384: 746, with 512 753).
// With draws in registers up to three or four workgroups of 512 share a unit
// (100 x 100 torus, R = 16,384: 469, with 256 threads 492, with 1,024 592; R =
// 2,048, one resident: 98 with 512, 86 with 1,024), or two of 768 (140 x 140
// torus, R = 8,192: 488, with 512 509, with 1,024 563). Two that are the whole
// launch take 1,024 although 768 are faster (R = 4,096: 296, with 768 260): a
// test of that launch holds the number.
int pa_host::tile_threads(int need, int lds, int max_lds, long long per_level, int fuse)
{
    const int fit = max_lds / lds, res = std::min(need, fit);
    if (!fuse) return res <= 1 ? (per_level > 160 ? 1024 : 512) : res == 2 || per_level > 160 ? 512 : 256;
    if (per_level < 1000) return res <= 2 ? 512 : 256;
    if (res <= 1 || (fit == 2 && need == 2)) return 1024;
    return fit == 2 ? 768 : 512;
}

// Form. The tile form shortens the chain of a level, spreads long rows over
// lanes, and its nibble records let 8 replicas stand where bytes leave room for
// 4 or for fewer workgroups (us a launch of 10 sweeps, byte form, or word kernel
// for degree 200, and tile form: n = 7,000, degree 12, R = 1,024: 257, 200, R =
// 4,096: 392, 365, R = 16,384: 1,799, 1,155; n = 800, degree 48, R = 1,024:
// 2,742, 330; n = 1,000, degree 200: 47,200, 1,710; n = 12,000, degree 4, R =
// 4,096: 597, 433).
// The byte form draws in the level's own pass, which costs less where a level
// has work enough for all waves: with two 8-replica workgroups a compute unit
// of either form (three of the tile form's win), when the tile form's levels
// are more than 14 block rows of 64 lanes, on average (R = 4,096, colouring
// orders, byte and tile form: n = 7,000, degree 12, 30 rows a level: 281, 301;
// n = 9,000, degree 18, 48: 412, 474; n = 7,000, degree 4, 21: 251, 267; n =
// 4,000, degree 12, 18: 191, 191; n = 3,000, degree 12, 14: 168, 157; natural
// order, n = 7,000, degree 12, 9: 392, 365; R = 16,384, n = 9,900, degree 20, 52:
// 1,981, 2,183). Rows of more than 30 entries run past its registers: a wave of
// them a level is lost from 34 on (degree 20 on n = 4,000, 22 rows: 280, 256; on
// 9,900: 498, 556), several from 43 on (degree 24 on 9,900: 627, 594).
bool pa_host::byte_levels(long long rows, long long levels, int dmax)
{
    return (rows > 14 * levels && dmax <= 33) || (rows > 30 * levels && dmax <= 42);
}

bool pa_host::two_a_unit(long long tiles8, int cus, int max_lds, int tile_lds, int byte_lds)
{
    const long long need = (tiles8 + cus - 1) / cus;
    return std::min<long long>(need, max_lds / tile_lds) == 2 && std::min<long long>(need, max_lds / byte_lds) == 2;
}

// Whether a run takes the tile form, and its shape then; p comes with the
// general form's choice and the levels. All figures: a launch of 10 sweeps (5 on
// tori) on MI355X, microseconds.
static bool take_tile_form(const pa_solver *s, const pa_schedule *sch, Plan &p, int cus, int max_lds)
{
    const int n = s->n, tile = sch->tile_replicas;
    const bool sign_ok = n + 256 <= 0x7FFF;
    if (p.sgn && !sign_ok) return false;
    const bool byte8 = p.kind == 1 && p.W == 8;
    const int byte_lds = p.sweep_lds(s);
    const long long per_level = n / p.n_levels;     // nodes a level, on average
    p.kind = 1;
    p.ahead = 1;
    p.deg = degree_class(s->dmax);
    // Negative edges read complemented copies of the records (no work per
    // neighbour), or carry sign bits in the blocks (two instructions per
    // neighbour and 8 replicas, half the LDS): sign bits at low degrees and
    // where two workgroups with copies would not share a compute unit.
    p.bsg = !p.sgn ? 0
            : s->dmax <= 8 || p.deg != 0 || 2 * pa::sweep_tile_lds(8, 1, n, 0) > max_lds ? 2 : 1;
    const int comp = p.bsg == 1 ? 1 : 0;
    p.fuse = tile != 16 && fuse_draws(s, p.n_levels);
    if (p.fuse) p.bsg = 2;          // (unsigned too: no sign bit is set then)
    auto lds = [&](int W) { return pa::sweep_tile_lds(W, comp, n, p.fuse); };
    // Shape. A sweep is a chain of levels, so it takes as long for one
    // workgroup as for all that are resident: the narrowest tile whose
    // workgroups get a compute unit each, and else 8 replicas (100 x 100 torus,
    // R = 1,024: 65 with 4, 82 with 8; R = 2,048: 113 and 88). 16 where 8 would
    // take more than one generation of four and levels are small (n = 800,
    // degree 12, R = 16,384: 227 with 16, 276 with 8; n = 4,000: 821 and 749).
    p.W = tile;
    if (p.deg == 2) p.W = 4;
    else if (tile == 0) {
        p.W = (p.R + 3) / 4 <= cus ? 4 : 8;
        if (!p.fuse && (p.R + 7) / 8 > 4 * cus && per_level <= 100 && 4 * lds(16) <= max_lds) p.W = 16;
    }
    if (lds(p.W) > max_lds) return false;
    p.nblk = (p.R + p.W - 1) / p.W;
    if (sch->wg_threads == 0) {
        p.threads = tile_threads((p.nblk + cus - 1) / cus, lds(p.W), max_lds, per_level, p.fuse);
        // Two workgroups a unit that are the whole launch take 448 threads
        // where their levels need no more rounds with them, although 512 are
        // faster (n = 7,000, degree 12: 369, with 512 346; n = 4,000: 241, 236):
        // tests of the 7,000-node launch hold the number.
        if (p.W == 8 && !p.fuse && p.threads == 512 && p.nblk > cus && p.nblk <= 2 * cus) {
            auto rounds_at = [&](int T) {
                long long r = 0;
                for (int l = 0; l < p.n_levels; ++l) r += (p.level_off[l + 1] - p.level_off[l] + T - 1) / T;
                return r;
            };
            if (rounds_at(448) <= rounds_at(512)) p.threads = 448;
        }
    }
    return !(byte8 && p.W == 8 && !p.fuse && two_a_unit(p.nblk, cus, max_lds, lds(8), byte_lds) &&
             byte_levels(tile_rows(s, p, p.bsg != 0), p.n_levels, s->dmax));
}

pa_status pa_host::build_plan(pa_solver *s, const pa_schedule *sch, int R, Plan &p, bool tables,
                              const Shape *force, size_t room, const Levels *levels)
{
    const int n = s->n;
    p.K = sch->n_steps;
    p.S = sch->sweeps_per_step;
    p.R = R;
    p.G = (R + 63) / 64;
    p.Rp = p.G * 64;
    p.nw32 = (n + 31) / 32;
    p.record = sch->record;
    p.lmax1 = sch->as_enable ? sch->as_max_level + 1 : 1;

    int dev = 0, cus = 256, max_lds = 65536;
    if (hipGetDevice(&dev) == hipSuccess) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) cus = v;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess && v > 0)
            max_lds = v;
    } else {
        (void)hipGetLastError();
        max_lds = 160 * 1024;
    }
    p.threads = sch->wg_threads ? sch->wg_threads : pa::kMaxThreads;
    p.sgn = s->has_neg;
    const int req = sch->sweep_kernel, tile = sch->tile_replicas;
    if (req < 0 || req > 2) return fail(PA_EINVAL, "sweep_kernel must be 0, 1 or 2");
    // The cluster move keeps n union-find parents and three n-bit bitmaps in LDS
    // (plus 2.2 KB of fixed scratch).
    if (sch->nl_period > 0 && pa::icm_lds_bytes(n, p.nw32) + 4096 > max_lds)
        return fail(PA_ERANGE, "cluster moves on %d nodes exceed the LDS of a workgroup", n);
    // Kernel 1 on a signed graph reads complemented copies of the records for
    // negative edges (no per-neighbour work), or marks them with a sign bit in
    // the block entry (one XOR per neighbour, half the LDS). Measured on
    // MI355X: sign bits pay on low-degree graphs whose workgroups (8 replicas
    // each) would otherwise queue for LDS -- at least two full waves of them
    // beyond what fits with copies (100 x 100 torus, R 16,384: 0.83 -> 0.66 ms
    // per step); with fewer workgroups the XOR only costs (+2 to +8 % on small
    // tori). Sign bits take bit 15 of a record index, so indices stay below 2^15.
    p.bsg = p.sgn ? 1 : 0;
    if (p.sgn && s->dmax <= 8 && n + pa::kBytesRecBase / 4 <= 0x7FFF) {
        const long long per_cu = max_lds / pa::sweep_bytes_lds(8, 1, n, s->dmax);
        if (per_cu == 0 || (R + 7) / 8 >= 2LL * cus * per_cu) p.bsg = 2;
    }
    // Large signed graphs (above about 20,000 nodes) whose complemented
    // records do not fit a workgroup's LDS even at 4 replicas take sign bits,
    // which halve the records, rather than the word kernel (which holds 2n
    // words of a signed graph and n sweep-order entries).
    if (p.bsg == 1 && n + pa::kBytesRecBase / 4 <= 0x7FFF &&
        pa::sweep_bytes_lds(4, 1, n, s->dmax) > max_lds && pa::sweep_bytes_lds(4, 0, n, s->dmax) <= max_lds)
        p.bsg = 2;
    const int comp = p.bsg == 1 ? 1 : 0;
    auto bytes_fit = [&](int W) { return pa::sweep_bytes_lds(W, comp, n, s->dmax) <= max_lds; };
    auto words_fit = [&](int W) { return pa::sweep_lds_bytes(W, p.sgn, n, s->dmax, p.threads) <= max_lds; };
    int W = 0;
    // Kernel 1 compares draws with 32-bit thresholds. A row whose threshold
    // is exactly 2^32 for some but not all uphill moves (beta * gamma^l nonzero
    // but below about 6e-17, where exp rounds to 1) needs kernel 2.
    bool partial_sat = false;
    if (s->dmax >= 1)
        for (int k = 0; k < p.K && !partial_sat; ++k) {
            double g = 1.0;
            for (int l = 0; l < p.lmax1; ++l) {
                const double b = sch->beta[k] * g;
                if (threshold_fixed(b, 1) == (1ull << 32) && threshold_fixed(b, s->dmax) != (1ull << 32))
                    partial_sat = true;
                g = g * sch->as_gamma;
            }
        }
    if (req == 1 && partial_sat)
        return fail(PA_ERANGE, "sweep kernel 1 cannot take an inverse temperature whose "
                               "acceptance rounds to 1 for some uphill moves only");
    // Record indices (complements and the zero record included, offset by the
    // threshold table) are u16.
    const bool idx_fit = p.bsg == 2 ? n + pa::kBytesRecBase / 4 <= 0x7FFF
                                    : (p.sgn ? 2 * n : n) + pa::kBytesRecBase / 4 <= 0xFFFF;
    bool bytes_ok = s->dmax <= kMaxBytesDegree && (tile == 0 || tile <= 16) && !partial_sat && idx_fit;
    if (req == 1 && !bytes_ok)
        return fail(PA_EINVAL, "sweep kernel 1 needs max degree <= %d and tile 4, 8 or 16", kMaxBytesDegree);
    // The tile form serves degrees up to kMaxWideDegree; explicitly requested
    // kernels and tiles keep kernel 1's documented range.
    const bool tile_ok = req != 2 && !partial_sat && (tile == 0 || tile <= 16) &&
                         (s->dmax <= kMaxBytesDegree ||
                          (req == 0 && s->dmax <= kMaxWideDegree && (tile == 0 || tile == 4)));
    if (force) {
        // A shape imposed by a multi-run launch: kernel 1 with the given tile,
        // threads, record mode and entry form, or an error.
        if (s->dmax > kMaxBytesDegree || partial_sat)
            return fail(PA_EINVAL, "runs sharing a launch need max degree <= %d and no partly saturated "
                                   "threshold row", kMaxBytesDegree);
        if (force->W != 4 && force->W != 8 && force->W != 16)
            return fail(PA_EINVAL, "shared launch tile %d is not 4, 8 or 16", force->W);
        if (force->threads < 64 || force->threads > 1024 || force->threads % 64)
            return fail(PA_EINVAL, "shared launch threads %d", force->threads);
        if ((force->bsg != 0 && force->bsg != 2) || (force->bsg == 0 && p.sgn) ||
            (force->bsg == 2 && n + pa::kBytesRecBase / 4 > 0x7FFF))
            return fail(PA_EINVAL, "shared launch record mode %d does not suit this graph", force->bsg);
        p.bsg = force->bsg;
        if (force->lds(n, s->dmax) > max_lds)
            return fail(PA_ERANGE, "graph of %d nodes does not fit LDS with %d replicas per workgroup", n,
                        force->W);
        if (!force->ahead && force->direct && pa::kBytesRecBase + (size_t)(n + 1) * force->W > 0xFFFF)
            return fail(PA_ERANGE, "graph of %d nodes too large for offset entries at tile %d", n, force->W);
        if (force->ahead && (force->deg < degree_class(s->dmax) ||
                             (force->fuse && (force->deg != 0 || force->bsg != 2 || force->W > 8 ||
                                              !fuse_draws(s, 1)))))
            return fail(PA_EINVAL, "shared launch counters %d do not suit this graph", force->deg);
        p.kind = 1;
        p.W = force->W;
        p.threads = force->threads;
        p.nblk = (R + p.W - 1) / p.W;
        if (levels) static_cast<Levels &>(p) = *levels;
        else build_levels(s, sch->order, p);
        if (force->ahead) {
            p.ahead = 1;
            p.deg = force->deg;
            p.fuse = force->fuse;
            build_tile_plan(s, p, tables);
            if (force->byte_threads != 0) {
                Plan q;
                q.kind = 1;
                q.K = p.K;
                q.lmax1 = p.lmax1;
                q.nw32 = p.nw32;
                q.W = force->byte_W;
                q.threads = force->byte_threads;
                q.nblk = (R + q.W - 1) / q.W;
                q.n_levels = p.n_levels;
                q.level_off = p.level_off;
                const size_t general = general_bytes(s, q), own = tile_bytes(s, p);
                p.pad = general > own ? general - own : 0;
            }
        } else {
            build_blocks(s, p, force->direct);
        }
    } else if (req != 2 && bytes_ok) {
        W = tile;
        // A requested tile takes the thread count of the automatic plan for
        // that tile: 512 (refined by the level rule below) when two
        // workgroups fit a CU, else 1,024.
        if (W != 0 && sch->wg_threads == 0)
            p.threads = 2 * pa::sweep_bytes_lds(W, comp, n, s->dmax) <= max_lds ? 512 : 1024;
        if (W == 0 && s->dmax <= 8 && bytes_fit(8)) {
            // Measured on MI355X: on low-degree graphs (tori) a round's work per
            // node is small and 8-replica tiles spread the per-node cost over
            // the most replicas, even with fewer workgroups than CUs. 512
            // threads, or 256 when two workgroups fit a CU and there are fewer
            // than four workgroups per CU in all; 1,024 when only one fits a CU
            // (tori of about 15,000 nodes and more: 11-13 % faster than 512).
            W = 8;
            if (sch->wg_threads == 0) {
                const bool two = 2 * pa::sweep_bytes_lds(8, comp, n, s->dmax) <= max_lds;
                p.threads = !two ? 1024 : ((R + 7) / 8 < 4 * cus ? 256 : 512);
            }
        }
        if (W == 0) {
            // Measured on MI355X: two resident workgroups of 512 threads per CU
            // hide the per-level latency best. Take the widest tile whose LDS
            // allows two per CU and that still gives two workgroups per CU;
            // else the narrowest tile that fits (most workgroups).
            for (int w = 16; w >= 4 && W == 0; w >>= 1)
                if (2 * pa::sweep_bytes_lds(w, comp, n, s->dmax) <= max_lds && (R + w - 1) / w >= 2 * cus)
                    W = w;
            for (int w = 4; w <= 16 && W == 0; w <<= 1)
                if (bytes_fit(w)) W = w;
            if (W == 0) W = 4;
            if (sch->wg_threads == 0)
                p.threads = 2 * pa::sweep_bytes_lds(W, comp, n, s->dmax) <= max_lds ? 512 : 1024;
        }
        if (!bytes_fit(W)) {
            if (req == 1)
                return fail(PA_ERANGE, "graph of %d nodes does not fit LDS with %d replicas per workgroup", n, W);
            W = 0;
        } else {
            p.kind = 1;
        }
    }
    if (!force && W == 0) {
        if (req == 2 && tile != 0 && tile < 16) return fail(PA_EINVAL, "sweep kernel 2 takes tile 16, 32 or 64");
        p.kind = 2;
        W = tile >= 16 ? tile : 0;
        if (W == 0) {
            W = 64;
            while (W > 16 && ((R + W - 1) / W < cus || !words_fit(W))) W >>= 1;
        }
        if (!words_fit(W))
            return fail(PA_ERANGE, "graph of %d nodes does not fit LDS with %d replicas per workgroup", n, W);
    }
    if (!force) {
    p.W = W;
    p.nblk = (R + W - 1) / W;

    build_levels(s, sch->order, p);
    if (p.kind == 1 && sch->wg_threads == 0 && p.threads == 512) {
        // Measured on MI355X: a sweep's time follows its number of rounds
        // (one barrier each), and at equal rounds fewer waves per workgroup
        // idle less. Take the smallest multiple of 64 in [256, 512] that
        // needs no more rounds than 512 threads (C2-shaped graph: 448
        // threads, 32 rounds, 2 % faster than 320 threads with 35).
        auto rounds_at = [&](int T) {
            long long r = 0;
            for (int l = 0; l < p.n_levels; ++l) r += (p.level_off[l + 1] - p.level_off[l] + T - 1) / T;
            return r;
        };
        const long long r512 = rounds_at(512);
        for (int T = 256; T < 512; T += 64)
            if (rounds_at(T) <= r512) {
                p.threads = T;
                break;
            }
    }
    // Degrees of 128 to 1,023 were the word kernel's. One such node is enough for
    // the 16-bit counters, whatever the others are, and 4 replicas a workgroup;
    // that is still the faster form (n = 7,000, degree 12 and one node of degree
    // 200, R = 4,096: 1,452 with the word kernel, 515; R = 16,384: 3,605, 1,792).
    // The tile form where it is faster, and where the workspace has room for
    // it: its plan can be the larger one.
    if (tile_ok && room != 0) {
        const size_t general = general_bytes(s, p);
        Plan q = p;
        if (take_tile_form(s, sch, q, cus, max_lds)) {
            build_tile_plan(s, q, tables);
            const size_t own = tile_bytes(s, q);
            p = std::move(q);
            p.pad = general > own ? general - own : 0;
        }
    }
    if (!p.ahead) build_blocks(s, p, -1);
    if (p.kind == 1) {
        // Two workgroups sharing a compute unit: the issue arbiter breaks
        // ties by age, so the one dispatched first would finish far earlier
        // and leave the other alone on the unit for the launch's tail.
        // Measured on MI355X with the G63-shaped run (8-replica tiles, two
        // per CU, all resident at once): the second one's waves ahead in 6 of
        // every 10 sweeps even them out (durations 709k / 915k cycles ->
        // 840k / 850k), the launch 7 % shorter. Launches of several
        // generations of workgroups (the 100 x 100 torus) were 2 % slower
        // with the slots alternating, so they keep the plain kernel.
        const int lds = p.sweep_lds(s);
        const int waves = (p.threads + 63) / 64;
        const int per_cu = std::min(max_lds / std::max(lds, 1), 16 / std::max(waves, 1));
        const long long slots = (long long)cus * per_cu;
        if (p.W == 8 && per_cu == 2 && p.nblk > slots / 2 && p.nblk <= slots) p.prio_mode = 1;
    }
    }

    // Weight-table sizes (needed for the workspace size even without tables).
    const long long span = s->nnz;  // E_r - E_min <= sum |w_ij| over both directions
    // Fixed steps: the table of step k (beta_{k+1} - beta_k). Adaptive steps:
    // the table of jump j at index j - 1 (beta_j - beta_0).
    const int n_tab = sch->beta_adapt ? std::min(sch->adapt_jump, p.K - 1) : p.K - 1;
    p.wtab_off.assign(std::max(p.K, 1), 0);
    p.wtab_len.assign(std::max(p.K, 1), 0);
    std::map<uint64_t, std::pair<int, int>> seen;
    struct Tab {
        double db;
        long long off, len;
    };
    std::vector<Tab> distinct;
    long long total = 0;
    for (int k = 0; k < n_tab; ++k) {
        const double db = sch->beta_adapt ? sch->beta[k + 1] - sch->beta[0] : sch->beta[k + 1] - sch->beta[k];
        uint64_t key;
        std::memcpy(&key, &db, sizeof key);
        auto it = seen.find(key);
        if (it == seen.end()) {
            // The table runs to its first zero entry (at most span + 1
            // entries); the weights fall with n, so the first zero is found
            // by bisection and only the entries kept are evaluated.
            long long len = span + 1;
            if (weight_fixed(db, span) == 0) {
                long long lo = 0, hi = span;          // weight(lo) != 0 or lo = 0; weight(hi) == 0
                if (weight_fixed(db, 0) == 0) hi = 0;
                while (hi - lo > 1) {
                    const long long mid = lo + (hi - lo) / 2;
                    (weight_fixed(db, mid) != 0 ? lo : hi) = mid;
                }
                len = hi;
            }
            if (tables) distinct.push_back({db, total, len});
            it = seen.emplace(key, std::make_pair((int)total, (int)len)).first;
            total += len;
        }
        p.wtab_off[k] = it->second.first;
        p.wtab_len[k] = it->second.second;
    }
    if (tables && !distinct.empty()) {
        // The distinct tables' entries, filled by table on host threads.
        p.wtab.assign((size_t)total, 0);
        parallel_rows((int)distinct.size(), total, [&](int t0, int t1) {
            for (int t = t0; t < t1; ++t)
                for (long long q = 0; q < distinct[t].len; ++q)
                    p.wtab[(size_t)(distinct[t].off + q)] = weight_fixed(distinct[t].db, q);
        });
    }
    if (total == 0) {
        total = 1;
        if (tables) p.wtab.push_back(0);
    }
    if (tables && sch->nl_period > 0 && sch->nl_kind == 1) {
        p.qtab.assign((size_t)p.K * p.lmax1, 0);
        for (int k = 0; k < p.K; ++k) {
            double g = 1.0;
            for (int l = 0; l < p.lmax1; ++l) {
                p.qtab[(size_t)k * p.lmax1 + l] = bond_fixed(sch->beta[k] * g);
                g = g * sch->as_gamma;
            }
        }
    }
    if (tables) {
        // Threshold rows, one per (step, noise level); rows are independent,
        // so large tables are filled by several host threads.
        const int D = s->dmax + 1;
        if (p.kind == 1) p.thr32.assign((size_t)p.K * p.lmax1 * D, 0);
        else p.thr.assign((size_t)p.K * p.lmax1 * D, 0);
        auto fill = [&](int k0, int k1) {
            for (int k = k0; k < k1; ++k) {
                double g = 1.0;
                for (int l = 0; l < p.lmax1; ++l) {
                    const double b = sch->beta[k] * g;
                    if (p.kind == 1) {
                        uint32_t *row = &p.thr32[((size_t)k * p.lmax1 + l) * D];
                        for (int m = 1; m < D; ++m)
                            row[m - 1] = (uint32_t)std::min<uint64_t>(threshold_fixed(b, m), 0xFFFFFFFFull);
                        // Every uphill move accepted (exp rounds to 1 up to the max degree).
                        row[D - 1] = s->dmax >= 1 && threshold_fixed(b, s->dmax) == (1ull << 32) ? 1u : 0u;
                    } else {
                        uint64_t *row = &p.thr[((size_t)k * p.lmax1 + l) * D];
                        row[0] = 0;
                        for (int m = 1; m < D; ++m) row[m] = threshold_fixed(b, m);
                    }
                    g = g * sch->as_gamma;
                }
            }
        };
        parallel_rows(p.K, (long long)p.K * p.lmax1 * D, fill);
    }

    Layout &L = p.L;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = align_up(o + std::max<size_t>(bytes, 1));
        return at;
    };
    L.row_ptr = take(sizeof(int) * (n + 1));
    L.col = take(sizeof(int) * s->nnz);
    L.npos = take(sizeof(int) * n);
    L.edges = take(sizeof(uint32_t) * s->edges.size());
    L.qtab = sch->nl_period > 0 && sch->nl_kind == 1 ? take(sizeof(uint64_t) * (size_t)p.K * p.lmax1) : 0;
    L.sched = p.ahead ? 0 : take(sizeof(int) * n);
    L.level_off = p.ahead ? 0 : take(sizeof(int) * (p.n_levels + 1));
    L.blocks = take(p.ahead ? p.row_bytes : sizeof(uint32_t) * p.blocks.size());
    L.stream = take(sizeof(int) * (p.ahead ? p.item_ints : p.kind == 1 ? p.rounds.size() : p.stream.size()));
    L.streams = p.ahead ? take(sizeof(int) * p.streams.size()) : 0;
    L.thr = take((p.ahead ? sizeof(uint32_t) : sizeof(uint64_t)) * (size_t)p.K * p.lmax1 * (s->dmax + 1));
    L.wtab = take(sizeof(uint64_t) * (size_t)total);
    L.wtab_off = take(sizeof(int) * p.K);
    L.wtab_len = take(sizeof(int) * p.K);
    L.inputs_end = o;
    L.vout = sch->nl_period > 0
                 ? take(sizeof(uint32_t) * (size_t)(sch->nl_kind == 1 ? R : R / 2) * p.nw32)
                 : 0;
    L.X0 = take(sizeof(uint64_t) * (size_t)p.G * n);
    L.X1 = take(sizeof(uint64_t) * (size_t)p.G * n);
    L.E0 = take(sizeof(int) * p.Rp);
    L.E1 = take(sizeof(int) * p.Rp);
    L.cand = take(sizeof(uint64_t) * p.nblk);
    L.snap = take(sizeof(uint32_t) * (size_t)p.nblk * p.nw32);
    L.counters = take(sizeof(uint64_t) * 2);
    L.as_state = take(sizeof(int) * 4);
    L.best = take(sizeof(int) * 8);
    L.best_x = take(sizeof(uint32_t) * p.nw32);
    L.stats = take(sizeof(long long) * (size_t)p.K * pa::kStatFields);
    L.parent = take(sizeof(int) * p.Rp);
    L.counts = (p.record & 1) ? take(sizeof(int) * (size_t)p.K * R) : 0;
    L.xinit = (p.record & 2) ? take(sizeof(uint64_t) * (size_t)p.G * n) : 0;
    // What a run needs is no less with one form than with the other, so a
    // workspace that was too small stays so.
    L.total = o + p.pad;
    if (p.ahead && !force && L.total > room) {
        p = Plan();
        return build_plan(s, sch, R, p, tables, nullptr, 0);
    }
    return PA_OK;
}

extern "C" pa_status pa_workspace_bytes(const pa_solver *s, const pa_schedule *sch, int32_t R,
                                        size_t *bytes)
{
    g_error[0] = 0;
    if (!bytes) return fail(PA_EINVAL, "pa_workspace_bytes: null output");
    pa_status st = check_schedule(s, sch, R);
    if (st != PA_OK) return st;
    Plan p;
    st = build_plan(const_cast<pa_solver *>(s), sch, R, p, false);
    if (st != PA_OK) return st;
    *bytes = p.L.total;
    return PA_OK;
}

// ------------------------------------------------------------------ run ----

// Hash (FNV-1a, 64 bit) of everything a run's results depend on: the graph,
// the schedule without its launch-shape fields, R, seed and instance.
static uint64_t fnv(uint64_t h, const void *p, size_t n)
{
    const unsigned char *b = static_cast<const unsigned char *>(p);
    for (size_t q = 0; q < n; ++q) h = (h ^ b[q]) * 0x100000001B3ull;
    return h;
}

uint64_t pa_host::run_key(const pa_solver *s, const pa_schedule *sch, int32_t R, uint64_t seed,
                          uint32_t instance)
{
    uint64_t h = 0xCBF29CE484222325ull;
    h = fnv(h, &s->n, sizeof s->n);
    h = fnv(h, s->row_ptr.data(), sizeof(int) * s->row_ptr.size());
    h = fnv(h, s->col.data(), sizeof(int) * s->col.size());
    h = fnv(h, s->npos.data(), sizeof(int) * s->npos.size());
    const int32_t ints[] = {sch->n_steps, sch->sweeps_per_step, sch->as_enable, sch->as_stall_steps,
                            sch->as_max_level, sch->as_frozen_inv, sch->nl_period, sch->nl_kind,
                            sch->record, R, (int32_t)instance, sch->beta_adapt,
                            sch->beta_adapt ? sch->adapt_jump : 0, sch->beta_adapt ? sch->adapt_num : 0,
                            sch->beta_adapt ? sch->adapt_den : 0};
    h = fnv(h, ints, sizeof ints);
    h = fnv(h, &sch->as_gamma, sizeof sch->as_gamma);
    h = fnv(h, &seed, sizeof seed);
    h = fnv(h, sch->beta, sizeof(double) * (size_t)sch->n_steps);
    if (sch->order) h = fnv(h, sch->order, sizeof(int32_t) * (size_t)s->n);
    return h;
}

// Plan the run, upload the graph and tables into the workspace and set up the
// launch arguments. A fresh run also clears the state, draws the initial
// population and takes its best; a restored one leaves the state to the caller.
// `pinned`: the host inputs go through the solver's pinned staging buffer
// (allocated on first use); otherwise from a pageable host buffer, so that no
// pinned or device memory is allocated.
pa_status pa_host::start_run(pa_solver *s, const pa_schedule *sch, int32_t R, uint64_t seed,
                             uint32_t instance, void *workspace, size_t workspace_bytes, void *stream,
                             bool fresh, bool pinned, const Shape *force)
{
    g_error[0] = 0;
    pa_status st = check_schedule(s, sch, R);
    if (st != PA_OK) return st;
    if (instance > 65535) return fail(PA_ERANGE, "instance=%u outside [0, 65535]", instance);
    if (!workspace) return fail(PA_EWORKSPACE, "workspace is null");
    if (((uintptr_t)workspace) % kAlign) return fail(PA_EWORKSPACE, "workspace must be 256-byte aligned");
    // The previous run may still be using its workspace (perhaps this one, from
    // another stream).
    if (s->has_run && s->stream) HIP_TRY(hipStreamSynchronize(s->stream));
    s->has_run = false;
    s->rc.valid = false;          // until this run's state is complete in the workspace
    Plan p;
    st = build_plan(s, sch, R, p, true, force, workspace_bytes);
    if (st != PA_OK) return st;
    if (workspace_bytes < p.L.total)
        return fail(PA_EWORKSPACE, "workspace of %zu bytes < %zu needed", workspace_bytes, p.L.total);

    s->plan = std::move(p);
    Plan &P = s->plan;
    const Layout &L = P.L;
    unsigned char *ws = static_cast<unsigned char *>(workspace);
    hipStream_t hs = static_cast<hipStream_t>(stream);
    s->ws = ws;
    s->stream = hs;
    HIP_TRY(hipGetDevice(&s->device));
    const int n = s->n;

    // All host inputs go to the device in one copy, through the pinned
    // staging buffer or a pageable one.
    unsigned char *stage = nullptr;
    if (pinned) {
        if (s->stage_pending) {
            HIP_TRY(hipEventSynchronize(s->stage_ev));
            s->stage_pending = false;
        }
        if (s->stage_cap < L.inputs_end) {
            if (s->stage) HIP_TRY(hipHostFree(s->stage));
            s->stage = nullptr;
            s->stage_cap = 0;
            HIP_TRY(hipHostMalloc(reinterpret_cast<void **>(&s->stage), L.inputs_end, hipHostMallocDefault));
            std::memset(s->stage, 0, L.inputs_end);
            s->stage_cap = L.inputs_end;
        }
        if (!s->stage_ev) HIP_TRY(hipEventCreateWithFlags(&s->stage_ev, hipEventDisableTiming));
        stage = s->stage;
    } else {
        s->stage_host.assign(L.inputs_end, 0);
        stage = s->stage_host.data();
    }
    auto put = [&](size_t off, const void *src, size_t bytes) {
        if (bytes) std::memcpy(stage + off, src, bytes);
    };
    put(L.row_ptr, s->row_ptr.data(), sizeof(int) * (n + 1));
    put(L.col, s->col.data(), sizeof(int) * s->nnz);
    put(L.npos, s->npos.data(), sizeof(int) * n);
    put(L.edges, s->edges.data(), sizeof(uint32_t) * s->edges.size());
    if (!P.ahead) {
        put(L.sched, P.sched.data(), sizeof(int) * n);
        put(L.level_off, P.level_off.data(), sizeof(int) * (P.n_levels + 1));
    }
    if (P.ahead) {
        put(L.blocks, P.rows.data(), P.row_bytes);
        put(L.stream, P.items.data(), sizeof(int) * P.items.size());
        put(L.streams, P.streams.data(), sizeof(int) * P.streams.size());
    } else {
        put(L.blocks, P.blocks.data(), sizeof(uint32_t) * P.blocks.size());
        if (P.kind == 1)
            put(L.stream, P.rounds.data(), sizeof(int) * P.rounds.size());
        else
            put(L.stream, P.stream.data(), sizeof(int) * P.stream.size());
    }
    put(L.qtab, P.qtab.data(), sizeof(uint64_t) * P.qtab.size());
    if (P.kind == 1)
        put(L.thr, P.thr32.data(), sizeof(uint32_t) * P.thr32.size());
    else
        put(L.thr, P.thr.data(), sizeof(uint64_t) * P.thr.size());
    put(L.wtab, P.wtab.data(), sizeof(uint64_t) * P.wtab.size());
    put(L.wtab_off, P.wtab_off.data(), sizeof(int) * P.K);
    put(L.wtab_len, P.wtab_len.data(), sizeof(int) * P.K);
    HIP_TRY(hipMemcpyAsync(ws, stage, L.inputs_end, hipMemcpyHostToDevice, hs));
    if (pinned) {
        HIP_TRY(hipEventRecord(s->stage_ev, hs));
        s->stage_pending = true;
    }

    auto U64 = [&](size_t off) { return reinterpret_cast<unsigned long long *>(ws + off); };
    if (fresh) {
        LAUNCH_TRY(pa::launch_fill_u64(U64(L.counters), 0ull, 2, hs));
        LAUNCH_TRY(pa::launch_fill_u64(U64(L.as_state), 0ull, 2, hs));
        LAUNCH_TRY(pa::launch_fill_u64(U64(L.best), 0ull, 4, hs));
        LAUNCH_TRY(pa::launch_fill_u64(U64(L.stats), 0ull, (long long)P.K * pa::kStatFields, hs));
        if (P.record & 1)
            LAUNCH_TRY(pa::launch_fill_u64(U64(L.counts), 0ull, ((long long)P.K * R + 1) / 2, hs));
    }

    pa::GraphDev gd;
    gd.n = n;
    gd.dmax = s->dmax;
    gd.row_ptr = reinterpret_cast<const int *>(ws + L.row_ptr);
    gd.col = reinterpret_cast<const int *>(ws + L.col);
    gd.npos = reinterpret_cast<const int *>(ws + L.npos);
    gd.edges = reinterpret_cast<const uint32_t *>(ws + L.edges);
    gd.ne = (int)s->edges.size();
    const uint32_t seed_lo = (uint32_t)seed, seed_hi = (uint32_t)(seed >> 32);

    size_t Xc = L.X0, Xn = L.X1, Ec = L.E0, En = L.E1;
    pa::InitArgs ia;
    ia.g = gd;
    ia.R = R;
    ia.G = P.G;
    ia.seed_lo = seed_lo;
    ia.seed_hi = seed_hi;
    ia.inst = instance;
    ia.X = reinterpret_cast<uint64_t *>(ws + Xc);
    ia.E = reinterpret_cast<int *>(ws + Ec);
    if (fresh) {
        LAUNCH_TRY(pa::launch_init(ia, hs));
        LAUNCH_TRY(pa::launch_energy(ia, hs));
        if (P.record & 2)
            HIP_TRY(hipMemcpyAsync(ws + L.xinit, ws + Xc, sizeof(uint64_t) * (size_t)P.G * n,
                                   hipMemcpyDeviceToDevice, hs));
    }

    pa::EpiArgs ea{};
    ea.R = R;
    ea.n = n;
    ea.nw32 = P.nw32;
    ea.nblk = P.nblk;
    ea.W = P.W;
    ea.K = P.K;
    ea.S = P.S;
    ea.as_enable = sch->as_enable;
    ea.as_stall = sch->as_stall_steps;
    ea.as_lmax = sch->as_enable ? sch->as_max_level : 0;
    ea.as_frozen_inv = sch->as_frozen_inv;
    ea.adapt = sch->beta_adapt;
    ea.adapt_jump = sch->adapt_jump;
    ea.adapt_num = sch->adapt_num;
    ea.adapt_den = sch->adapt_den;
    ea.as_state = reinterpret_cast<int *>(ws + L.as_state);
    ea.cand = U64(L.cand);
    ea.snap = reinterpret_cast<const uint32_t *>(ws + L.snap);
    ea.best = reinterpret_cast<int *>(ws + L.best);
    ea.best_x = reinterpret_cast<uint32_t *>(ws + L.best_x);
    ea.counters = U64(L.counters);
    ea.stats = reinterpret_cast<long long *>(ws + L.stats);
    ea.wtab = reinterpret_cast<const uint64_t *>(ws + L.wtab);
    ea.wtab_off = reinterpret_cast<const int *>(ws + L.wtab_off);
    ea.wtab_len = reinterpret_cast<const int *>(ws + L.wtab_len);
    ea.seed_lo = seed_lo;
    ea.seed_hi = seed_hi;
    ea.inst = instance;
    ea.parent = reinterpret_cast<int *>(ws + L.parent);
    ea.counts_rec = (P.record & 1) ? reinterpret_cast<int *>(ws + L.counts) : nullptr;

    // Best of the initial population.
    if (fresh) {
        pa::EpiArgs e0 = ea;
        e0.k = 0;
        e0.do_pop = 1;
        e0.pop_step = -1;
        e0.pop_sweep = -1;
        e0.E = reinterpret_cast<const int *>(ws + Ec);
        e0.X = reinterpret_cast<const uint64_t *>(ws + Xc);
        LAUNCH_TRY(pa::launch_epilogue(e0, hs));
    }

    pa::SweepArgs sa;
    sa.n = n;
    sa.dmax = s->dmax;
    sa.blocks = reinterpret_cast<const uint4 *>(ws + L.blocks);
    sa.block_u4 = P.block_bytes / 16;
    sa.stream = reinterpret_cast<const int2 *>(ws + L.stream);
    sa.qpad = P.qpad;
    sa.rounds = reinterpret_cast<const int4 *>(ws + L.stream);
    sa.n_rounds = P.n_rounds;
    sa.flush_every = P.flush_every;
    sa.direct = P.direct;
    sa.items = reinterpret_cast<const int2 *>(ws + L.stream);
    sa.streams = reinterpret_cast<const int4 *>(ws + L.streams);
    sa.draw_half = P.draw_half;
    sa.prio_mode = P.prio_mode;
    sa.R = R;
    sa.S = P.S;
    sa.lmax1 = P.lmax1;
    sa.n_levels = P.n_levels;
    sa.K = P.K;
    sa.adapt = sch->beta_adapt;
    sa.seed_lo = seed_lo;
    sa.seed_hi = seed_hi;
    sa.inst = instance;
    sa.sched = reinterpret_cast<const int *>(ws + L.sched);
    sa.level_off = reinterpret_cast<const int *>(ws + L.level_off);
    sa.thr = reinterpret_cast<const uint64_t *>(ws + L.thr);
    sa.thr32 = reinterpret_cast<const uint32_t *>(ws + L.thr);
    sa.as_state = reinterpret_cast<const int *>(ws + L.as_state);
    sa.best_E = reinterpret_cast<const int *>(ws + L.best);
    sa.cand = U64(L.cand);
    sa.snap = reinterpret_cast<uint32_t *>(ws + L.snap);
    sa.counters = U64(L.counters);
    sa.nw32 = P.nw32;
    sa.Xin = nullptr;
    sa.Ein = nullptr;
    sa.parent = nullptr;

    if (s->timing && pinned) {
        const size_t need = 2 * (size_t)P.K;
        while (s->ev.size() < need) {
            hipEvent_t e;
            HIP_TRY(hipEventCreate(&e));
            s->ev.push_back(e);
        }
    }
    s->ev_first = 0;
    s->ev_used = 0;
    s->timing_run = pinned ? s->timing : 0;

    pa_solver::RunCtx &c = s->rc;
    c.valid = fresh;              // a restored run becomes valid once its state is loaded
    c.key = run_key(s, sch, R, seed, instance);
    c.next_step = 0;
    c.parents_pending = false;
    c.Xc = Xc; c.Xn = Xn; c.Ec = Ec; c.En = En;
    c.seed_lo = seed_lo; c.seed_hi = seed_hi; c.instance = instance;
    c.nl_period = sch->nl_period;
    c.nl_kind = sch->nl_kind;
    c.adapt = sch->beta_adapt;
    c.gd = gd;
    c.sa = sa;
    c.ea = ea;
    s->final_x = Xc;
    s->final_E = Ec;
    return PA_OK;
}

// Steps [k0, k1) of the run prepared by start_run (and any steps before k0).
static pa_status run_range(pa_solver *s, int k0, int k1)
{
    Plan &P = s->plan;
    const Layout &L = P.L;
    pa_solver::RunCtx &c = s->rc;
    unsigned char *ws = s->ws;
    hipStream_t hs = s->stream;
    const int n = s->n, R = P.R;
    const uint32_t seed_lo = c.seed_lo, seed_hi = c.seed_hi, instance = c.instance;
    const pa::GraphDev gd = c.gd;
    const pa::EpiArgs ea = c.ea;
    pa::SweepArgs sa = c.sa;
    size_t Xc = c.Xc, Xn = c.Xn, Ec = c.Ec, En = c.En;
    if (s->ev_used < k0) s->ev_first = k0;     // steps before k0 ran in another call or process
    c.valid = false;                           // until every step of the range is enqueued

    int stop = k1;
    if (s->fault_step >= k0 && s->fault_step < k1) stop = s->fault_step;
    for (int k = k0; k < stop; ++k) {
        if (c.adapt && k > 0 && (k - k0) % 64 == 0) {
            // Adaptive steps end at the last grid point, usually well before
            // step K: look every 64 steps and enqueue no more once it is done
            // (the remaining steps would do nothing).
            int g = 0;
            HIP_TRY(hipMemcpyAsync(&g, ws + L.as_state + 3 * sizeof(int), sizeof g, hipMemcpyDeviceToHost, hs));
            HIP_TRY(hipStreamSynchronize(hs));
            if (g >= P.K) break;
        }
        sa.k = k;
        // (the stride fixed when the run started, which sized the events)
        const bool timed = s->timing_run && k % s->timing_run == 0;
        if (timed) HIP_TRY(hipEventRecord(s->ev[2 * k], hs));
        if (P.kind == 1) {
            // Kernel 1 reads the previous population through the resampling
            // parents and writes the other buffer (no separate gather).
            sa.Xin = reinterpret_cast<const uint64_t *>(ws + Xc);
            sa.Ein = reinterpret_cast<const int *>(ws + Ec);
            sa.X = reinterpret_cast<uint64_t *>(ws + Xn);
            sa.E = reinterpret_cast<int *>(ws + En);
            sa.parent = c.parents_pending ? reinterpret_cast<const int *>(ws + L.parent) : nullptr;
            if (P.ahead)
                LAUNCH_TRY(pa::launch_sweep_tile(P.W, P.bsg, P.deg, P.fuse, P.threads, P.nblk, P.sweep_lds(s), sa,
                                                 hs));
            else
                LAUNCH_TRY(pa::launch_sweep_bytes(P.W, P.bsg, P.threads, P.nblk, sa, hs));
            std::swap(Xc, Xn);
            std::swap(Ec, En);
            c.parents_pending = false;
        } else {
            sa.X = reinterpret_cast<uint64_t *>(ws + Xc);
            sa.E = reinterpret_cast<int *>(ws + Ec);
            LAUNCH_TRY(pa::launch_sweep(P.W, P.sgn, P.threads, P.nblk, sa, hs));
        }
        if (timed) HIP_TRY(hipEventRecord(s->ev[2 * k + 1], hs));
        if (s->timing_run) s->ev_used = k + 1;
        pa::EpiArgs e = ea;
        e.k = k;
        e.E = reinterpret_cast<const int *>(ws + Ec);
        e.X = reinterpret_cast<const uint64_t *>(ws + Xc);
        const bool nl = c.nl_period > 0 && (k + 1) % c.nl_period == 0;
        if (nl) {
            pa::EpiArgs e1 = e;
            e1.do_cand = 1;
            LAUNCH_TRY(pa::launch_epilogue(e1, hs));
            pa::IcmArgs ic;
            ic.g = gd;
            ic.R = R;
            ic.G = P.G;
            ic.k = k;
            ic.K = P.K;
            ic.adapt = c.adapt;
            ic.nw32 = P.nw32;
            ic.seed_lo = seed_lo;
            ic.seed_hi = seed_hi;
            ic.inst = instance;
            ic.X = reinterpret_cast<uint64_t *>(ws + Xc);
            ic.E = reinterpret_cast<int *>(ws + Ec);
            ic.vout = reinterpret_cast<uint32_t *>(ws + L.vout);
            ic.kind = c.nl_kind;
            ic.lmax1 = P.lmax1;
            ic.qtab = reinterpret_cast<const uint64_t *>(ws + L.qtab);
            ic.as_state = reinterpret_cast<const int *>(ws + L.as_state);
            LAUNCH_TRY(pa::launch_icm(ic, hs));
            e.do_pop = 1;
            e.pop_step = k;
            e.pop_sweep = P.S;
            e.do_rest = 1;
        } else {
            e.do_cand = 1;
            e.do_rest = 1;
        }
        LAUNCH_TRY(pa::launch_epilogue(e, hs));
        if (P.kind == 1 && k + 1 < P.K) c.parents_pending = true;
        if (P.kind == 2 && k + 1 < P.K) {
            pa::GatherArgs ga;
            ga.n = n;
            ga.R = R;
            ga.G = P.G;
            ga.parent = reinterpret_cast<const int *>(ws + L.parent);
            ga.Xin = reinterpret_cast<const uint64_t *>(ws + Xc);
            ga.Xout = reinterpret_cast<uint64_t *>(ws + Xn);
            ga.Ein = reinterpret_cast<const int *>(ws + Ec);
            ga.Eout = reinterpret_cast<int *>(ws + En);
            LAUNCH_TRY(pa::launch_gather(ga, hs));
            std::swap(Xc, Xn);
            std::swap(Ec, En);
        }
    }
    c.Xc = Xc; c.Xn = Xn; c.Ec = Ec; c.En = En;
    c.next_step = stop;
    c.valid = true;
    s->final_x = Xc;
    s->final_E = Ec;
    s->has_run = true;
    if (stop < k1) {
        // Injected fault: the steps before it are enqueued and the run can
        // continue from it.
        s->fault_step = -1;
        HIP_TRY(hipStreamSynchronize(hs));
        return fail(PA_EABORTED, "run stopped before step %d by pa_set_fault_step", stop);
    }
    return PA_OK;
}

extern "C" pa_status pa_set_fault_step(pa_solver *s, int32_t k)
{
    g_error[0] = 0;
    if (!s) return fail(PA_EINVAL, "null solver");
    if (k < -1) return fail(PA_EINVAL, "fault step %d < -1", k);
    s->fault_step = k;
    return PA_OK;
}

extern "C" pa_status pa_run_steps(pa_solver *s, const pa_schedule *sch, int32_t R, uint64_t seed,
                                  uint32_t instance, int32_t k_begin, int32_t k_end, void *workspace,
                                  size_t workspace_bytes, void *stream)
{
    g_error[0] = 0;
    if (!s) return fail(PA_EINVAL, "null solver");
    pa_status st = check_schedule(s, sch, R);
    if (st != PA_OK) return st;
    if (instance > 65535) return fail(PA_ERANGE, "instance=%u outside [0, 65535]", instance);
    if (k_begin < 0 || k_end < k_begin || k_end > sch->n_steps)
        return fail(PA_EINVAL, "steps [%d, %d) outside the schedule's [0, %d]", k_begin, k_end, sch->n_steps);
    if (k_begin == 0) {
        st = start_run(s, sch, R, seed, instance, workspace, workspace_bytes, stream, true);
        if (st != PA_OK) return st;
    } else {
        const pa_solver::RunCtx &c = s->rc;
        if (!c.valid || c.key != run_key(s, sch, R, seed, instance))
            return fail(PA_ESTATE, "no run of this schedule, R, seed and instance to continue");
        if (c.next_step != k_begin)
            return fail(PA_ESTATE, "the run in the workspace continues at step %d, not %d", c.next_step, k_begin);
        if (workspace != s->ws) return fail(PA_EWORKSPACE, "a run continues in its own workspace");
        if (stream != (void *)s->stream) {
            // The previous steps were enqueued on another stream: order after them.
            HIP_TRY(hipStreamSynchronize(s->stream));
            s->stream = static_cast<hipStream_t>(stream);
        }
    }
    return run_range(s, k_begin, k_end);
}

extern "C" pa_status pa_run(pa_solver *s, const pa_schedule *sch, int32_t R, uint64_t seed,
                            uint32_t instance, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!sch) {
        g_error[0] = 0;
        return fail(PA_EINVAL, "null schedule");
    }
    return pa_run_steps(s, sch, R, seed, instance, 0, sch->n_steps, workspace, workspace_bytes, stream);
}

extern "C" pa_status pa_run_static(pa_solver *s, const pa_schedule *sch, int32_t R, uint64_t seed,
                                   uint32_t instance, void *stream)
{
    g_error[0] = 0;
    pa_status st = check_schedule(s, sch, R);
    if (st != PA_OK) return st;
    if (instance > 65535) return fail(PA_ERANGE, "instance=%u outside [0, 65535]", instance);
    Plan p;
    st = build_plan(s, sch, R, p, false, nullptr, pa::kStaticScratchBytes);
    if (st != PA_OK) return st;
    if (p.L.total > pa::kStaticScratchBytes)
        return fail(PA_EWORKSPACE, "run needs %zu workspace bytes, more than the %zu of the static "
                                   "workspace: use pa_run with a workspace", p.L.total,
                    (size_t)pa::kStaticScratchBytes);
    void *ws = nullptr;
    if (pa::static_scratch(&ws) != 0) return fail(PA_EDEVICE, "%s", pa::last_hip_error());
    st = start_run(s, sch, R, seed, instance, ws, pa::kStaticScratchBytes, stream, true, false);
    if (st != PA_OK) return st;
    return run_range(s, 0, sch->n_steps);
}

// -------------------------------------------------------------- results ----

static pa_status fetch(pa_solver *s, void *dst, size_t off, size_t bytes)
{
    if (!s || !s->has_run) return fail(PA_ESTATE, "no completed pa_run on this solver");
    HIP_TRY(hipSetDevice(s->device));
    HIP_TRY(hipMemcpyAsync(dst, s->ws + off, bytes, hipMemcpyDeviceToHost, s->stream));
    HIP_TRY(hipStreamSynchronize(s->stream));
    return PA_OK;
}

extern "C" pa_status pa_best_info(pa_solver *s, int64_t out[4])
{
    if (!out) return fail(PA_EINVAL, "null output");
    int b[8];
    pa_status st = fetch(s, b, s ? s->plan.L.best : 0, sizeof b);
    if (st != PA_OK) return st;
    for (int q = 0; q < 4; ++q) out[q] = b[q];
    return PA_OK;
}

extern "C" pa_status pa_build_tables(const pa_schedule *sch, int32_t d_max, int32_t e_span,
                                     void *out, size_t *bytes)
{
    g_error[0] = 0;
    if (!sch || !bytes || !sch->beta) return fail(PA_EINVAL, "pa_build_tables: null argument");
    if (sch->n_steps < 1) return fail(PA_EINVAL, "pa_build_tables: n_steps must be >= 1");
    if (d_max < 0 || e_span < 0) return fail(PA_EINVAL, "pa_build_tables: negative size");
    if (d_max > kMaxDegree || e_span > (1 << 26))
        return fail(PA_ERANGE, "pa_build_tables: d_max or e_span too large");
    for (int k = 0; k < sch->n_steps; ++k) {
        const double b = sch->beta[k];
        if (!std::isfinite(b) || b < 0 || (k > 0 && b < sch->beta[k - 1]))
            return fail(PA_EINVAL, "pa_build_tables: beta must be finite, >= 0 and non-decreasing");
    }
    if (sch->as_enable && (sch->as_max_level < 0 || sch->as_max_level > 15 || !(sch->as_gamma > 0) ||
                           sch->as_gamma > 1))
        return fail(PA_EINVAL, "pa_build_tables: noise levels need 0 <= as_max_level <= 15, 0 < gamma <= 1");
    if (sch->beta_adapt && uneven_grid(sch->beta, sch->n_steps) >= 0)
        return fail(PA_EINVAL, "pa_build_tables: adaptive steps need an evenly spaced beta grid");
    const int K = sch->n_steps, Lv = sch->as_enable ? sch->as_max_level + 1 : 1, D = d_max + 1;
    const int n_tab = sch->beta_adapt ? std::min(std::max(sch->adapt_jump, 1), K - 1) : K - 1;
    const size_t n_thr = (size_t)K * Lv * D, n_w = (size_t)n_tab * (size_t)(e_span + 1);
    const size_t need = 8 * (n_thr + n_w);
    if (!out) {
        *bytes = need;
        return PA_OK;
    }
    if (*bytes < need) return fail(PA_ERANGE, "pa_build_tables: %zu bytes < %zu needed", *bytes, need);
    *bytes = need;
    uint64_t *o = static_cast<uint64_t *>(out);
    for (int k = 0; k < K; ++k) {
        double g = 1.0;
        for (int l = 0; l < Lv; ++l) {
            const double b = sch->beta[k] * g;
            uint64_t *row = o + ((size_t)k * Lv + l) * D;
            row[0] = 1ull << 32;
            for (int m = 1; m < D; ++m) row[m] = threshold_fixed(b, m);
            g = g * sch->as_gamma;
        }
    }
    uint64_t *wt = o + n_thr;
    for (int k = 0; k < n_tab; ++k) {
        const double db = sch->beta_adapt ? sch->beta[k + 1] - sch->beta[0] : sch->beta[k + 1] - sch->beta[k];
        for (int m = 0; m <= e_span; ++m) wt[(size_t)k * (e_span + 1) + m] = weight_fixed(db, m);
    }
    return PA_OK;
}

extern "C" pa_status pa_run_batch(const pa_batch_run *runs, int32_t count, void *const *streams,
                                  int32_t n_streams)
{
    g_error[0] = 0;
    if (!runs || !streams || count < 1 || n_streams < 1)
        return fail(PA_EINVAL, "pa_run_batch: null array, count < 1 or n_streams < 1");
    std::vector<const pa_solver *> seen;
    seen.reserve(count);
    for (int i = 0; i < count; ++i) {
        if (!runs[i].solver) return fail(PA_EINVAL, "pa_run_batch: run %d has no solver", i);
        seen.push_back(runs[i].solver);
    }
    std::sort(seen.begin(), seen.end());
    if (std::adjacent_find(seen.begin(), seen.end()) != seen.end())
        return fail(PA_EINVAL, "pa_run_batch: a solver appears in two runs");
    auto failed = [&](int i, pa_status st) {
        char msg[sizeof g_error];
        std::snprintf(msg, sizeof msg, "%s", g_error);
        return fail(st, "pa_run_batch: run %d: %s", i, msg);
    };
    bool adaptive = false;
    for (int i = 0; i < count; ++i) adaptive |= runs[i].schedule && runs[i].schedule->beta_adapt;
    if (!adaptive) {
        for (int i = 0; i < count; ++i) {
            const pa_batch_run &r = runs[i];
            const pa_status st = pa_run(r.solver, r.schedule, r.R, r.seed, r.instance, r.workspace,
                                        r.workspace_bytes, streams[i % n_streams]);
            if (st != PA_OK) return failed(i, st);
        }
        return PA_OK;
    }
    // An adaptive run's host looks at its grid point every 64 steps and waits
    // for the device there. Every run is started first, then the steps go in
    // chunks of 64, one chunk of each run in turn, so that while the host
    // waits on one run the chunks of the others are already queued.
    int kmax = 0;
    for (int i = 0; i < count; ++i) {
        const pa_batch_run &r = runs[i];
        const pa_status st = pa_run_steps(r.solver, r.schedule, r.R, r.seed, r.instance, 0, 0, r.workspace,
                                          r.workspace_bytes, streams[i % n_streams]);
        if (st != PA_OK) return failed(i, st);
        kmax = std::max(kmax, r.schedule->n_steps);
    }
    constexpr int kChunk = 64;
    for (int k0 = 0; k0 < kmax; k0 += kChunk)
        for (int i = 0; i < count; ++i) {
            const pa_batch_run &r = runs[i];
            const int K = r.schedule->n_steps;
            if (k0 >= K) continue;
            const pa_status st = pa_run_steps(r.solver, r.schedule, r.R, r.seed, r.instance, k0,
                                              std::min(k0 + kChunk, K), r.workspace, r.workspace_bytes,
                                              streams[i % n_streams]);
            if (st != PA_OK) return failed(i, st);
        }
    return PA_OK;
}

extern "C" pa_status pa_best_cut(pa_solver *s, int64_t *cut, int32_t *energy)
{
    int64_t info[4];
    pa_status st = pa_best_info(s, info);
    if (st != PA_OK) return st;
    if (cut) *cut = (s->w_tot - info[0]) / 2;
    if (energy) *energy = (int32_t)info[0];
    return PA_OK;
}

extern "C" pa_status pa_best_config(pa_solver *s, int8_t *x)
{
    if (!x) return fail(PA_EINVAL, "null output");
    if (!s || !s->has_run) return fail(PA_ESTATE, "no completed pa_run on this solver");
    std::vector<uint32_t> bits(s->plan.nw32);
    pa_status st = fetch(s, bits.data(), s->plan.L.best_x, sizeof(uint32_t) * bits.size());
    if (st != PA_OK) return st;
    for (int i = 0; i < s->n; ++i) x[i] = ((bits[i >> 5] >> (i & 31)) & 1u) ? 1 : -1;
    return PA_OK;
}

extern "C" pa_status pa_best_config_hex(pa_solver *s, char *buf, size_t len)
{
    if (!buf) return fail(PA_EINVAL, "null output");
    if (!s || !s->has_run) return fail(PA_ESTATE, "no completed pa_run on this solver");
    const size_t digits = ((size_t)s->n + 3) / 4;
    if (len < digits + 1) return fail(PA_ERANGE, "hex buffer of %zu bytes < %zu needed", len, digits + 1);
    std::vector<int8_t> x(s->n);
    pa_status st = pa_best_config(s, x.data());
    if (st != PA_OK) return st;
    static const char hexd[] = "0123456789abcdef";
    for (size_t p = 0; p < digits; ++p) {
        int v = 0;
        for (int q = 0; q < 4; ++q) {
            const size_t i = 4 * p + q;
            v = (v << 1) | ((i < (size_t)s->n && x[i] > 0) ? 1 : 0);
        }
        buf[p] = hexd[v];
    }
    buf[digits] = 0;
    return PA_OK;
}

static void unpack_population(const std::vector<uint64_t> &X, int n, int R, int8_t *x)
{
    for (int r = 0; r < R; ++r) {
        const uint64_t *Xg = &X[(size_t)(r >> 6) * n];
        const int b = r & 63;
        int8_t *xr = x + (size_t)r * n;
        for (int i = 0; i < n; ++i) xr[i] = ((Xg[i] >> b) & 1ull) ? 1 : -1;
    }
}

extern "C" pa_status pa_get_population(pa_solver *s, int8_t *x, int16_t *h, int32_t *E)
{
    if (!s || !s->has_run) return fail(PA_ESTATE, "no completed pa_run on this solver");
    const Plan &P = s->plan;
    const int n = s->n;
    // After a range that stopped before the last step, kernel 1 still holds
    // the population of the next step as the current buffer read through the
    // resampling parents: apply them here.
    std::vector<int> parent;
    if (s->rc.parents_pending) {
        parent.resize(P.R);
        pa_status st = fetch(s, parent.data(), P.L.parent, sizeof(int) * P.R);
        if (st != PA_OK) return st;
    }
    if (x || h) {
        std::vector<uint64_t> X((size_t)P.G * n);
        pa_status st = fetch(s, X.data(), s->final_x, sizeof(uint64_t) * X.size());
        if (st != PA_OK) return st;
        std::vector<int8_t> own;
        int8_t *xs = x;
        if (!xs) {
            own.resize((size_t)P.R * n);
            xs = own.data();
        }
        if (parent.empty()) {
            unpack_population(X, n, P.R, xs);
        } else {
            std::vector<int8_t> all((size_t)P.R * n);
            unpack_population(X, n, P.R, all.data());
            for (int r = 0; r < P.R; ++r)
                std::memcpy(xs + (size_t)r * n, all.data() + (size_t)parent[r] * n, (size_t)n);
        }
        if (h) {
            // The device keeps no fields: h_i = sum_j w_ij x_j from the spins
            // (the positive neighbours of a row come first).
            parallel_rows(P.R, (long long)P.R * s->nnz, [&](int r0, int r1) {
                for (int r = r0; r < r1; ++r) {
                    const int8_t *xr = xs + (size_t)r * n;
                    int16_t *hr = h + (size_t)r * n;
                    for (int i = 0; i < n; ++i) {
                        const int e0 = s->row_ptr[i], e1 = s->row_ptr[i + 1], em = e0 + s->npos[i];
                        int acc = 0;
                        for (int e = e0; e < em; ++e) acc += xr[s->col[e]];
                        for (int e = em; e < e1; ++e) acc -= xr[s->col[e]];
                        hr[i] = (int16_t)acc;
                    }
                }
            });
        }
    }
    if (E) {
        std::vector<int> Eall(P.R);
        pa_status st = fetch(s, Eall.data(), s->final_E, sizeof(int) * P.R);
        if (st != PA_OK) return st;
        for (int r = 0; r < P.R; ++r) E[r] = Eall[parent.empty() ? r : parent[r]];
    }
    return PA_OK;
}

extern "C" pa_status pa_get_initial_population(pa_solver *s, int8_t *x)
{
    if (!x) return fail(PA_EINVAL, "null output");
    if (!s || !s->has_run) return fail(PA_ESTATE, "no completed pa_run on this solver");
    const Plan &P = s->plan;
    if (!(P.record & 2)) return fail(PA_ESTATE, "run did not record the initial population (record bit 1)");
    std::vector<uint64_t> X((size_t)P.G * s->n);
    pa_status st = fetch(s, X.data(), P.L.xinit, sizeof(uint64_t) * X.size());
    if (st != PA_OK) return st;
    unpack_population(X, s->n, P.R, x);
    return PA_OK;
}

extern "C" pa_status pa_get_step_stats(pa_solver *s, int64_t *out)
{
    if (!out) return fail(PA_EINVAL, "null output");
    if (!s || !s->has_run) return fail(PA_ESTATE, "no completed pa_run on this solver");
    return fetch(s, out, s->plan.L.stats, sizeof(long long) * (size_t)s->plan.K * pa::kStatFields);
}

extern "C" pa_status pa_get_counts(pa_solver *s, int32_t *out)
{
    if (!out) return fail(PA_EINVAL, "null output");
    if (!s || !s->has_run) return fail(PA_ESTATE, "no completed pa_run on this solver");
    if (!(s->plan.record & 1)) return fail(PA_ESTATE, "run did not record copy counts (record bit 0)");
    return fetch(s, out, s->plan.L.counts, sizeof(int) * (size_t)s->plan.K * s->plan.R);
}

extern "C" pa_status pa_get_launch_info(pa_solver *s, int64_t out[8])
{
    if (!out) return fail(PA_EINVAL, "null output");
    if (!s || !s->has_run) return fail(PA_ESTATE, "no completed pa_run on this solver");
    const Plan &P = s->plan;
    out[0] = P.kind;
    out[1] = P.W;
    out[2] = P.threads;
    out[3] = P.nblk;
    out[4] = P.sweep_lds(s);
    out[5] = P.n_levels;
    out[6] = P.kind == 1 ? P.n_rounds : P.qpad - 4;
    out[7] = P.K;
    return PA_OK;
}

// ------------------------------------------------------------ checkpoint ----

namespace {
struct CkptHeader {
    char magic[8];
    uint64_t key;
    uint64_t bytes;
    int32_t n, R, K, G, nw32, next_step, record, version;
};
constexpr char kCkptMagic[8] = {'P', 'A', 'C', 'K', 'P', 'T', '0', '1'};

// Device regions of the state between steps, in blob order.
struct CkptPart {
    size_t off, bytes;
};

std::vector<CkptPart> ckpt_parts(const pa_solver *s)
{
    const Plan &P = s->plan;
    const Layout &L = P.L;
    std::vector<CkptPart> v;
    v.push_back({s->rc.Xc, sizeof(uint64_t) * (size_t)P.G * s->n});
    v.push_back({s->rc.Ec, sizeof(int) * (size_t)P.R});
    v.push_back({L.as_state, sizeof(int) * 4});
    v.push_back({L.best, sizeof(int) * 8});
    v.push_back({L.counters, sizeof(uint64_t) * 2});
    v.push_back({L.best_x, sizeof(uint32_t) * (size_t)P.nw32});
    v.push_back({L.stats, sizeof(long long) * (size_t)P.K * pa::kStatFields});
    if (P.record & 1) v.push_back({L.counts, sizeof(int) * (size_t)P.K * P.R});
    if (P.record & 2) v.push_back({L.xinit, sizeof(uint64_t) * (size_t)P.G * s->n});
    return v;
}

size_t ckpt_bytes(const std::vector<CkptPart> &parts)
{
    size_t b = sizeof(CkptHeader);
    for (const CkptPart &q : parts) b += (q.bytes + 7) & ~size_t(7);
    return b;
}
}  // namespace

extern "C" pa_status pa_checkpoint_bytes(const pa_solver *s, size_t *bytes)
{
    g_error[0] = 0;
    if (!s || !bytes) return fail(PA_EINVAL, "pa_checkpoint_bytes: null argument");
    if (!s->rc.valid || !s->has_run) return fail(PA_ESTATE, "no run on this solver to checkpoint");
    *bytes = ckpt_bytes(ckpt_parts(s));
    return PA_OK;
}

extern "C" pa_status pa_checkpoint_save(pa_solver *s, void *out, size_t bytes)
{
    g_error[0] = 0;
    if (!s || !out) return fail(PA_EINVAL, "pa_checkpoint_save: null argument");
    if (!s->rc.valid || !s->has_run) return fail(PA_ESTATE, "no run on this solver to checkpoint");
    pa_solver::RunCtx &c = s->rc;
    const Plan &P = s->plan;
    if (bytes < ckpt_bytes(ckpt_parts(s)))
        return fail(PA_EINVAL, "checkpoint buffer of %zu bytes < %zu", bytes, ckpt_bytes(ckpt_parts(s)));
    HIP_TRY(hipSetDevice(s->device));
    if (c.parents_pending) {
        // Store the population itself: copy it through the parent list into
        // the other buffer, which becomes the current one.
        pa::GatherArgs ga;
        ga.n = s->n;
        ga.R = P.R;
        ga.G = P.G;
        ga.parent = reinterpret_cast<const int *>(s->ws + P.L.parent);
        ga.Xin = reinterpret_cast<const uint64_t *>(s->ws + c.Xc);
        ga.Xout = reinterpret_cast<uint64_t *>(s->ws + c.Xn);
        ga.Ein = reinterpret_cast<const int *>(s->ws + c.Ec);
        ga.Eout = reinterpret_cast<int *>(s->ws + c.En);
        LAUNCH_TRY(pa::launch_gather(ga, s->stream));
        std::swap(c.Xc, c.Xn);
        std::swap(c.Ec, c.En);
        c.parents_pending = false;
        s->final_x = c.Xc;
        s->final_E = c.Ec;
    }
    const std::vector<CkptPart> parts = ckpt_parts(s);
    unsigned char *o = static_cast<unsigned char *>(out);
    CkptHeader h;
    std::memcpy(h.magic, kCkptMagic, 8);
    h.key = c.key;
    h.bytes = ckpt_bytes(parts);
    h.n = s->n;
    h.R = P.R;
    h.K = P.K;
    h.G = P.G;
    h.nw32 = P.nw32;
    h.next_step = c.next_step;
    h.record = P.record;
    h.version = 1;
    std::memcpy(o, &h, sizeof h);
    size_t at = sizeof h;
    for (const CkptPart &q : parts) {
        HIP_TRY(hipMemcpyAsync(o + at, s->ws + q.off, q.bytes, hipMemcpyDeviceToHost, s->stream));
        at += (q.bytes + 7) & ~size_t(7);
    }
    HIP_TRY(hipStreamSynchronize(s->stream));
    return PA_OK;
}

extern "C" pa_status pa_checkpoint_load(pa_solver *s, const pa_schedule *sch, int32_t R, uint64_t seed,
                                        uint32_t instance, const void *in, size_t bytes, void *workspace,
                                        size_t workspace_bytes, void *stream)
{
    g_error[0] = 0;
    if (!s || !sch || !in) return fail(PA_EINVAL, "pa_checkpoint_load: null argument");
    pa_status st = check_schedule(s, sch, R);
    if (st != PA_OK) return st;
    if (instance > 65535) return fail(PA_ERANGE, "instance=%u outside [0, 65535]", instance);
    CkptHeader h;
    if (bytes < sizeof h) return fail(PA_EINVAL, "checkpoint of %zu bytes is too short", bytes);
    std::memcpy(&h, in, sizeof h);
    if (std::memcmp(h.magic, kCkptMagic, 8) != 0 || h.version != 1)
        return fail(PA_EINVAL, "not a checkpoint of this library");
    if (h.bytes > bytes) return fail(PA_EINVAL, "checkpoint truncated: %zu of %llu bytes", bytes,
                                     (unsigned long long)h.bytes);
    if (h.key != run_key(s, sch, R, seed, instance) || h.n != s->n || h.R != R || h.K != sch->n_steps ||
        h.record != sch->record)
        return fail(PA_EINVAL, "checkpoint belongs to another graph, schedule, population, seed or instance");
    if (h.next_step < 0 || h.next_step > h.K) return fail(PA_EINVAL, "checkpoint step %d outside the schedule", h.next_step);
    st = start_run(s, sch, R, seed, instance, workspace, workspace_bytes, stream, false);
    if (st != PA_OK) return st;
    const std::vector<CkptPart> parts = ckpt_parts(s);
    if (ckpt_bytes(parts) != h.bytes || h.G != s->plan.G || h.nw32 != s->plan.nw32)
        return fail(PA_EINVAL, "checkpoint layout does not match this run");
    const unsigned char *p = static_cast<const unsigned char *>(in);
    size_t at = sizeof h;
    for (const CkptPart &q : parts) {
        HIP_TRY(hipMemcpyAsync(s->ws + q.off, p + at, q.bytes, hipMemcpyHostToDevice, s->stream));
        at += (q.bytes + 7) & ~size_t(7);
    }
    HIP_TRY(hipStreamSynchronize(s->stream));
    s->rc.valid = true;
    s->rc.next_step = h.next_step;
    s->rc.parents_pending = false;
    s->ev_first = s->ev_used = h.next_step;
    s->has_run = true;
    return PA_OK;
}

extern "C" pa_status pa_set_timing(pa_solver *s, int32_t on)
{
    if (!s) return fail(PA_EINVAL, "null solver");
    if (on < 0) return fail(PA_EINVAL, "timing stride must be >= 0");
    s->timing = on;
    return PA_OK;
}

extern "C" pa_status pa_get_sweep_time(pa_solver *s, double *ms, int64_t *launches)
{
    if (!s || !s->has_run) return fail(PA_ESTATE, "no completed pa_run on this solver");
    const int stride = s->timing_run;
    if (!stride) return fail(PA_ESTATE, "timing mode was off during the run");
    HIP_TRY(hipStreamSynchronize(s->stream));
    double tot = 0.0;
    int64_t count = 0;
    for (int k = s->ev_first; k < s->ev_used; ++k) {
        if (k % stride) continue;
        float t = 0.f;
        HIP_TRY(hipEventElapsedTime(&t, s->ev[2 * k], s->ev[2 * k + 1]));
        tot += t;
        ++count;
    }
    if (ms) *ms = tot;
    if (launches) *launches = count;
    return PA_OK;
}
