// Host side of the cache-blocked executor (see blocked.hpp): groups a fused
// list into segments, builds each gate's in-tile description, and queues the
// passes.
#include <algorithm>
#include <cstring>
#include <iterator>

#include "blocked.hpp"
#include "internal.hpp"

namespace cast {

struct BlockedPlan {
    int tb = 0, nt = 0;                // tile bits, workgroup size
    int knob_tb = 0, knob_mfma = 0, knob_3m = 0;   // tile groups: the knobs they were planned with
    struct Pass {
        size_t first = 0, count = 0;   // fused gates [first, first + count) covered by this pass
        bool segment = false;
        size_t gate = 0;               // ordinary pass: the fused gate it applies (a tile group's plan: the
                                       // schedule pass)
        BlkSeg seg{};
    };
    std::vector<Pass> passes;
    std::vector<BlkGate> gates;
    std::vector<BlkEnt> ent;           // of the operations
    std::vector<BlkEnt> units;         // work units of the table builds, behind them on the device
    std::vector<BlkMember> members;
    std::vector<double> tabs;          // phases of the diagonal gates (complex entries as pairs)
    void *dev = nullptr;               // device copy of these tables (phases in the state dtype)
    bool shares = false;               // it lies in the fused list's matrix block
    size_t dev_ent = 0, dev_mem = 0, dev_tabs = 0;   // byte offsets in it
};

void blocked_free(BlockedPlan *b) {
    if (!b) return;
    if (!b->shares) dev_free(b->dev);
    delete b;
}

namespace {

// Qubits mixed by a plan's blocks: the targets its first d virtual basis
// vectors touch.
uint64_t span_qubits(const PassPlan &p) {
    uint64_t m = 0;
    for (int i = 0; i < p.d; ++i)
        for (int s = 0; s < p.k; ++s)
            if ((p.L[i] >> s) & 1u) m |= 1ull << p.q[s];
    return m;
}

// Window w of a tile of 2^tb amplitudes that holds the qubits `need`: the
// fixed point of w = tb - #{q in need : q >= w}; false if it drops below the
// smallest window.
bool window_of(uint64_t need, int tb, int *w_out) {
    int w = tb;
    for (;;) {
        const int w2 = tb - __builtin_popcountll(need >> w);
        if (w2 < kBlkMinWindow) return false;
        if (w2 == w) break;
        w = w2;
    }
    *w_out = w;
    return true;
}

// LDS element of tile position y (as the kernel's at<S>, linear over GF(2)).
uint32_t lds_elem(uint32_t y, cast_dtype dt) {
    const uint32_t sh = dt == CAST_C128 ? 0 : 1, c = y >> sh;
    return ((c ^ (((c >> 4) ^ (c >> 8)) & 15u)) << sh) | (y & ((1u << sh) - 1));
}

// Index of qubit q in the tile number: the bits of the global index that are
// no tile bits, in order.
int tile_number_bit(int q, int w, const int *qh, int nh) {
    int b = q - w;
    for (int i = 0; i < nh; ++i) b -= qh[i] < q;
    return b;
}

// Appends n zeroed entries.
BlkEnt *append(std::vector<BlkEnt> *ent, uint32_t n) {
    ent->resize(ent->size() + n);
    return ent->data() + ent->size() - n;
}

BlkGate make_gate(const PassPlan &p, cast_dtype dt, int tb, int w, const int *qh, int nh, uint64_t mat,
                  std::vector<BlkEnt> *ent) {
    BlkGate g;
    std::memset(&g, 0, sizeof g);
    g.kind = 1;
    g.d = p.d;
    g.mat = mat;
    int tpos[kMaxK];   // tile bit of each target, -1: outside the tile
    for (int s = 0; s < p.k; ++s) {
        tpos[s] = p.q[s] < w ? p.q[s] : -1;
        for (int i = 0; i < nh; ++i)
            if (qh[i] == p.q[s]) tpos[s] = w + i;
    }
    // L^-1 by Gauss-Jordan: row r of [A | I] with A[r][c] = bit r of L[c]
    const int k = p.k;
    uint32_t rows[kMaxK];
    for (int r = 0; r < k; ++r) {
        rows[r] = 1u << (k + r);
        for (int c = 0; c < k; ++c)
            if ((p.L[c] >> r) & 1u) rows[r] |= 1u << c;
    }
    for (int c = 0; c < k; ++c) {
        int pr = c;
        while (!((rows[pr] >> c) & 1u)) ++pr;   // L is invertible
        std::swap(rows[c], rows[pr]);
        for (int r = 0; r < k; ++r)
            if (r != c && ((rows[r] >> c) & 1u)) rows[r] ^= rows[c];
    }
    // columns of L^-1: virtual coordinates of local index bit s
    uint32_t colv[kMaxK];
    for (int s = 0; s < k; ++s) {
        colv[s] = 0;
        for (int i = 0; i < k; ++i) colv[s] |= ((rows[i] >> (k + s)) & 1u) << i;
        if (tpos[s] >= 0) continue;
        for (int i = 0; i < k; ++i)
            if ((colv[s] >> i) & 1u) g.par[i] |= 1u << tile_number_bit(p.q[s], w, qh, nh);
    }
    // span offsets in tile coordinates (every span target is in the tile)
    uint32_t span[kGroupMaxD];
    for (int i = 0; i < p.d; ++i) {
        span[i] = 0;
        for (int s = 0; s < k; ++s)
            if ((p.L[i] >> s) & 1u) span[i] |= 1u << tpos[s];
        g.span[i] = lds_elem(span[i], dt);
    }
    // pivot bits of a reduced echelon basis of the span: the tile positions
    // with zeros there hold one element of every coset
    uint32_t b[kGroupMaxD];
    int piv[kGroupMaxD];
    for (int i = 0; i < p.d; ++i) {
        b[i] = span[i];
        for (int j = 0; j < i; ++j)
            if ((b[i] >> piv[j]) & 1u) b[i] ^= b[j];
        piv[i] = 31 - __builtin_clz(b[i]);
        for (int j = 0; j < i; ++j)
            if ((b[j] >> piv[i]) & 1u) b[j] ^= b[i];
    }
    for (uint32_t blk : p.blk) g.amask |= 1u << blk;
    // coset bits: the lane takes tile bits that are no targets (u is then the
    // same for the whole wave), spread over the LDS columns -- chunk bits i,
    // i + 4 and i + 8 share one (lds_elem) -- the wave and iteration the rest
    uint32_t targets = 0, pivots = 0, lane = 0;
    for (int s = 0; s < k; ++s)
        if (tpos[s] >= 0) targets |= 1u << tpos[s];
    for (int i = 0; i < p.d; ++i) pivots |= 1u << piv[i];
    int used[5] = {0, 0, 0, 0, 0};
    auto column = [&](int bit) { return dt == CAST_C128 ? bit & 3 : bit == 0 ? 4 : (bit - 1) & 3; };
    while (g.nlane < (p.d >= 4 ? 4u : 6u)) {
        int best = -1;
        for (int t = 0; t < tb; ++t)
            if (!(((targets | lane) >> t) & 1u) && (best < 0 || used[column(t)] < used[column(best)])) best = t;
        if (best < 0) break;
        lane |= 1u << best;
        ++used[column(best)];
        g.lane[g.nlane++] = lds_elem(1u << best, dt);
    }
    std::vector<int> rest;
    for (int t = 0; t < tb; ++t)
        if (!(((pivots | lane) >> t) & 1u)) rest.push_back(t);
    g.nuni = (uint32_t)rest.size();
    g.ent = (uint32_t)ent->size();
    // both parts are linear over GF(2): entry e from the one without its lowest bit
    BlkEnt *es = append(ent, 1u << g.nuni);
    for (uint32_t i = 0; i < g.nuni; ++i) {
        BlkEnt b{0, lds_elem(1u << rest[i], dt)};
        for (int s = 0; s < k; ++s)
            if (tpos[s] == rest[i]) b.u ^= colv[s];
        for (uint32_t e = 0; e < (1u << i); ++e) es[e | 1u << i] = BlkEnt{es[e].u ^ b.u, es[e].a ^ b.a};
    }
    return g;
}

// A stretch of diagonal gates as phase tables over tile bits: gates join a
// table while its tile bits stay within kBlkTabBits (first fit; diagonal
// gates commute).
struct Cluster {
    std::vector<int> bits;                    // tile bits, ascending
    std::vector<const PhaseTable *> gates;
};
std::vector<Cluster> cluster_tables(const std::vector<PhaseTable> &tabs, const int *pos) {
    std::vector<Cluster> out;
    for (const PhaseTable &t : tabs) {
        std::vector<int> in;
        for (int s = 0; s < t.k; ++s)
            if (pos[t.q[s]] >= 0) in.push_back(pos[t.q[s]]);
        std::sort(in.begin(), in.end());
        Cluster *to = nullptr;
        std::vector<int> u;
        for (Cluster &c : out) {
            u.clear();
            std::set_union(c.bits.begin(), c.bits.end(), in.begin(), in.end(), std::back_inserter(u));
            if ((int)u.size() <= std::max(kBlkTabBits, (int)in.size())) {
                to = &c;
                break;
            }
        }
        if (!to) {
            out.emplace_back();
            to = &out.back();
            u = in;
        }
        to->bits = u;
        to->gates.push_back(&t);
    }
    return out;
}

// Appends the segment that applies the (non-identity) gates `cur`, fused gates
// [first, first + count), whose mixed qubits `need` fit a tile.
void emit_segment(BlockedPlan *bp, const std::vector<PassPlan> &P, const std::vector<size_t> &off, int n,
                  cast_dtype dt, const std::vector<size_t> &cur, size_t first, size_t count, uint64_t need) {
    const int tb = bp->tb;
    const size_t ab = amp_bytes(dt);
    size_t mats = 0, area = 0;
    for (size_t i : cur) {
        if (P[i].d >= 4) mats += (P[i].blk.size() * ab) << (2 * P[i].d);
        if (P[i].d == 0) area = kBlkAreaBytes;
    }
    // with matrices in LDS: two workgroups where a compute unit holds both
    const size_t tile = ab << tb;
    const bool two = tile >= kBlkTileBytes / 2 && tile + mats + area <= kBlkMaxLds / 2;
    const int nt = !mats ? bp->nt : two ? 512 : kGroupThreads;
    int w = tb;
    window_of(need, tb, &w);
    BlockedPlan::Pass ps;
    ps.first = first, ps.count = count, ps.segment = true;
    BlkSeg &s = ps.seg;
    s.tb = tb, s.w = w, s.nh = 0;
    s.ntiles = 1ull << (n - tb);
    for (int q = w; q < n; ++q)
        if ((need >> q) & 1u) {
            s.qh[s.nh] = q;
            s.hlowmask[s.nh] = (1ull << q) - 1;
            ++s.nh;
        }
    s.g0 = (uint32_t)bp->gates.size();
    int pos[64];
    for (int q = 0; q < n; ++q) pos[q] = q < w ? q : -1;
    for (int i = 0; i < s.nh; ++i) pos[s.qh[i]] = w + i;
    uint32_t build = ~0u, used = 0;   // the open kind-2 operation, entries its tables take
    std::vector<PhaseTable> tabs;     // the open stretch of diagonal gates
    auto flush = [&] {
        const std::vector<Cluster> cl = cluster_tables(tabs, pos);
        for (size_t c = 0; c < cl.size();) {
            // a run: tables that fit the area together
            const size_t first_gate = bp->gates.size();
            std::vector<BlkGate> run;
            uint32_t end = used;
            bool fresh = build == ~0u;
            for (; c < cl.size() && run.size() < kBlkRunMax; ++c) {
                const uint32_t sz = 1u << cl[c].bits.size(), at = (end + sz - 1) & ~(sz - 1);
                if ((at + sz) * ab > kBlkAreaBytes) {
                    if (!run.empty()) break;
                    fresh = true;   // the area starts anew
                    end = 0;
                    --c;
                    continue;
                }
                BlkGate g;
                std::memset(&g, 0, sizeof g);
                g.k = (int)cl[c].bits.size();
                for (int i = 0; i < g.k; ++i) g.pos[i] = cl[c].bits[i];
                g.lds = at;
                end = at + sz;
                g.m0 = (uint32_t)bp->members.size();
                for (const PhaseTable *t : cl[c].gates) {
                    BlkMember m;
                    std::memset(&m, 0, sizeof m);
                    m.k = t->k;
                    m.tab = bp->tabs.size();
                    for (int i = 0; i < t->k; ++i) {
                        m.q[i] = t->q[i];
                        m.src[i] = pos[t->q[i]] < 0 ? -1
                            : (int)(std::lower_bound(cl[c].bits.begin(), cl[c].bits.end(), pos[t->q[i]]) - cl[c].bits.begin());
                    }
                    for (const cplx &z : t->ph) bp->tabs.push_back(z.real()), bp->tabs.push_back(z.imag());
                    bp->members.push_back(m);
                }
                g.m1 = (uint32_t)bp->members.size();
                run.push_back(g);
            }
            if (fresh) {
                build = (uint32_t)first_gate;
                BlkGate g;
                std::memset(&g, 0, sizeof g);
                g.kind = 2;
                bp->gates.push_back(g);
            }
            used = end;
            const uint32_t M = (uint32_t)run.size(), iters = std::max(1u, (1u << tb) / (uint32_t)nt);
            run[0].run = (int)M;
            run[0].ent = (uint32_t)bp->ent.size();
            BlkEnt *es = append(&bp->ent, iters * M);
            for (uint32_t it = 0; it < iters; ++it)
                for (uint32_t t = 0; t < M; ++t)
                    for (int i = 0; i < run[t].k; ++i)
                        es[it * M + t].u |= (((it * (uint32_t)nt) >> run[t].pos[i]) & 1u) << i;
            bp->gates.insert(bp->gates.end(), run.begin(), run.end());
            s.lds_tabs = std::max(s.lds_tabs, (uint32_t)(used * ab));
        }
        tabs.clear();
    };
    for (size_t i : cur) {
        if (P[i].d > 0) {
            flush();
            bp->gates.push_back(make_gate(P[i], dt, tb, w, s.qh, s.nh, off[i], &bp->ent));
            continue;
        }
        // neighbours are multiplied here while their union fits a
        // table of the host's size, which leaves fewer to build with
        PhaseTable t = phase_table(P[i]);
        if (tabs.empty() || !merge_tables(&tabs.back(), t, kRunMaxQ)) tabs.push_back(std::move(t));
    }
    flush();
    // the first tables are built at the start of the tile (nothing
    // reads the area before), and every build lists its units
    if (build != ~0u) {
        for (uint32_t gi = s.g0; gi < bp->gates.size(); ++gi)
            if (bp->gates[gi].kind == 2) {
                std::rotate(bp->gates.begin() + s.g0, bp->gates.begin() + gi, bp->gates.begin() + gi + 1);
                break;
            }
    }
    s.g1 = (uint32_t)bp->gates.size();
    for (uint32_t gi = s.g0; gi < s.g1; ++gi) {
        if (bp->gates[gi].kind != 2) continue;
        bp->gates[gi].ent = (uint32_t)bp->units.size();   // behind the operations' entries (upload_tables)
        for (uint32_t gj = gi + 1; gj < s.g1 && bp->gates[gj].kind != 2; ++gj)
            if (bp->gates[gj].kind == 0)
                for (uint32_t sl = 0; sl * 64 < (1u << bp->gates[gj].k); ++sl) bp->units.push_back(BlkEnt{gj, sl});
        bp->gates[gi].nent = (uint32_t)bp->units.size() - bp->gates[gi].ent;
    }
    s.nt = nt;
    s.lds_tabs = (s.lds_tabs + 15) & ~15u;
    for (uint32_t gi = s.g0; gi < s.g1; ++gi) {
        BlkGate &g = bp->gates[gi];
        if (g.kind != 1 || g.d < 4) continue;
        g.lds = s.lds_mats / (uint32_t)ab;
        s.lds_mats += (uint32_t)((size_t)__builtin_popcount(g.amask) * ab << (2 * g.d));
    }
    bp->passes.push_back(ps);
}

cast_status build(const cast_fused &f, cast_dtype dt, BlockedPlan **out) {
    const int tb = tuning().blocked_tile_bits[dt];
    if (((size_t)1 << tb) * amp_bytes(dt) > (64u << 10))
        return fail(CAST_EINVAL, "blocked_tile_bits: tile exceeds 64 KiB of LDS");
    auto *bp = new BlockedPlan;
    bp->tb = tb;
    bp->nt = blocked_threads(dt, tb);
    const int n = f.n;
    const std::vector<PassPlan> &P = f.plans;
    const std::vector<size_t> off = plan_offsets(P, dt);
    std::vector<size_t> cur;   // non-identity gates of the open segment
    size_t first = 0;
    uint64_t need = 0;
    auto close = [&](size_t end) {
        if (cur.size() == 1) {
            BlockedPlan::Pass ps;
            ps.first = first, ps.count = end - first, ps.gate = cur[0];
            bp->passes.push_back(ps);
        } else if (cur.size() > 1) {
            emit_segment(bp, P, off, n, dt, cur, first, end - first, need);
        }
        cur.clear();
        need = 0;
        first = end;
    };
    for (size_t i = 0; i < P.size(); ++i) {
        const PassPlan &p = P[i];
        if (p.identity()) continue;
        const uint64_t sp = span_qubits(p);
        int w;
        if (n < tb || p.d > kBlkMaxD || !window_of(sp, tb, &w)) {
            // an ordinary pass of its own
            close(i);
            BlockedPlan::Pass ps;
            ps.first = i, ps.count = 1, ps.gate = i;
            bp->passes.push_back(ps);
            first = i + 1;
            continue;
        }
        if (window_of(need | sp, tb, &w)) {
            need |= sp;
        } else {
            close(i);
            need = sp;
        }
        cur.push_back(i);
    }
    close(P.size());
    *out = bp;
    return CAST_OK;
}

// Uploads the list's matrices and the plan's tables, whichever are missing: a
// first call's in one allocation and one copy.
cast_status upload_tables(cast_fused *f, BlockedPlan *bp, cast_dtype dt) {
    const bool mats = !f->dev[dt].ptr && !f->plans.empty();
    if (bp->dev || bp->gates.empty())
        return mats ? upload_plans(f->plans, dt, &f->dev[dt], &f->dev_off[dt]) : CAST_OK;
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    bp->dev_ent = up(bp->gates.size() * sizeof(BlkGate));
    bp->dev_mem = bp->dev_ent + up((bp->ent.size() + bp->units.size() + kBlkEntsPad) * sizeof(BlkEnt));
    bp->dev_tabs = bp->dev_mem + up(bp->members.size() * sizeof(BlkMember));
    const size_t rsz = amp_bytes(dt) / 2, bytes = bp->dev_tabs + std::max<size_t>(bp->tabs.size(), 4) * rsz;
    auto write = [&](char *h) {
        for (size_t i = 0; i < bp->gates.size(); ++i) {
            BlkGate g = bp->gates[i];
            if (g.kind == 2) g.ent += (uint32_t)bp->ent.size();
            std::memcpy(h + i * sizeof g, &g, sizeof g);
        }
        BlkEnt *he = (BlkEnt *)(h + bp->dev_ent);
        std::copy(bp->ent.begin(), bp->ent.end(), he);
        std::copy(bp->units.begin(), bp->units.end(), he + bp->ent.size());
        if (!bp->members.empty())
            std::memcpy(h + bp->dev_mem, bp->members.data(), bp->members.size() * sizeof(BlkMember));
        for (size_t i = 0; i < bp->tabs.size(); ++i) {
            if (dt == CAST_C128) ((double *)(h + bp->dev_tabs))[i] = bp->tabs[i];
            else ((float *)(h + bp->dev_tabs))[i] = (float)bp->tabs[i];
        }
    };
    if (mats) {
        size_t at;
        if (cast_status rc = upload_plans(f->plans, dt, &f->dev[dt], &f->dev_off[dt], bytes, write, &at)) return rc;
        bp->dev = (char *)f->dev[dt].ptr + at;
        bp->shares = true;
        return CAST_OK;
    }
    std::vector<char> h(bytes);
    write(h.data());
    if (cast_status rc = dev_alloc(&bp->dev, bytes)) return rc;
    const hipError_t e = copy_to_device(bp->dev, h.data(), bytes);
    if (e != hipSuccess) {
        dev_free(bp->dev);
        bp->dev = nullptr;
        return fail(CAST_EHIP, std::string("blocked gate table upload: ") + hipGetErrorString(e));
    }
    return CAST_OK;
}

// The blocked grouping of a fused list for dtype dt (built on first use,
// rebuilt when the tile size knob has changed).  `device`: also upload the
// list's matrices and the grouping's gate table.
cast_status prepare(const cast_fused *fc, int n, cast_dtype dt, bool device, BlockedPlan **out) {
    if (!fc) return fail(CAST_EINVAL, "fused list is NULL");
    if (dt != CAST_C64 && dt != CAST_C128) return fail(CAST_EINVAL, "bad dtype");
    if (n != fc->n) return fail(CAST_EINVAL, "fused list was built for a different qubit count");
    cast_fused *f = const_cast<cast_fused *>(fc);
    BlockedPlan *&bp = f->blocked[dt];
    if (bp && (bp->tb != tuning().blocked_tile_bits[dt] || bp->nt != blocked_threads(dt, bp->tb))) {
        blocked_free(bp);
        bp = nullptr;
    }
    if (!bp) {
        if (cast_status rc = build(*f, dt, &bp)) return rc;
    }
    if (device)
        if (cast_status rc = upload_tables(f, bp, dt)) return rc;
    *out = bp;
    return CAST_OK;
}

cast_status launch_segment(cast_sv *sv, const cast_fused *f, const BlockedPlan &bp, const BlkSeg &seg) {
    const char *dev = static_cast<const char *>(bp.dev);
    const BlkPtrs ptrs{f->dev[sv->dt].ptr, dev + bp.dev_tabs, (const BlkGate *)dev, (const BlkEnt *)(dev + bp.dev_ent),
                       (const BlkMember *)(dev + bp.dev_mem)};
    return launch_blocked(sv->data, sv->dt, ptrs, seg, sv->stream);
}

cast_status launch(cast_sv *sv, const cast_fused *f, const BlockedPlan &bp, size_t i) {
    const BlockedPlan::Pass &ps = bp.passes[i];
    if (ps.segment) return launch_segment(sv, f, bp, ps.seg);
    const size_t rsz = sv->dt == CAST_C128 ? 8 : 4;
    const void *dm = (const char *)f->dev[sv->dt].ptr + f->dev_off[sv->dt][ps.gate] * rsz;
    return launch_pass(sv->data, sv->n, sv->dt, f->plans[ps.gate], dm, sv->stream);
}

cast_status check(const cast_sv *sv) {
    if (!sv || !sv->data) return fail(CAST_EINVAL, "state is NULL");
    return CAST_OK;
}

// ------------------------------------------------------------ tile groups
// apply_circuit's launches: consecutive passes of the schedule whose mixed
// qubits fit one LDS tile share a launch (and one read and write of the
// state) where that is predicted to be faster.  Times in microseconds, from
// kernel times at 12 to 26 qubits:
//   a pass    3.8 (direct, diagonal) to 6.5 (through LDS) on any small state,
//             then its bytes at 5.4 TB/s or its products at 60 / 120 TFLOP/s;
//   a group   5 (8 with tiles of 2^8 of a larger state, on 256 lanes: a
//             9-qubit Fourier transform fused to 6 qubits took 44.0 grouped
//             by 2^8, complex64, and takes 41.5 by 2^9) + the longer of the
//             state's read and write at 5.2 TB/s and its operations, + 0.3 of
//             the shorter (up to 256 tiles, a compute unit has one: their
//             sum, tile by tile at 0.1 TB/s, and operations but for the
//             matrix cores' take 1.2 as long).  An operation occupies a
//             compute unit for, per tile of 2^12 amplitudes: a table 0.3,
//             d = 1 0.7, d = 2 0.8, d = 3 1.1, and per tile of any size 0.1;
//             d = 4 / 5 3.0 / 5.3 (complex64: 1.5 / 2.8, matrix cores); never
//             less than 0.8, 1.6 or 2.6 (its barriers and first reads), nor
//             per tile than 0.55 of these for d = 4 and 5 (sixteen cosets are
//             a wave's: small tiles leave matrix cores idle).
struct Span {
    size_t a, b;          // schedule passes [a, b)
    uint64_t need;
    bool group;
};

// What the planning of every tile size asks of a schedule pass.
struct PassCost {
    bool live;            // not an identity
    bool mixes;           // has blocks of d >= 1
    int d;
    uint64_t span;        // qubits it mixes
    size_t mats;          // LDS bytes of its dense blocks
    double us;            // of its own launch
    double tabs;          // phase tables (diagonal run), else 1
};

std::vector<PassCost> pass_costs(const Schedule &sc, const std::vector<PassPlan> &P) {
    const double ab = (double)amp_bytes(sc.dt);
    std::vector<PassCost> out;
    out.reserve(sc.passes.size());
    for (const SchedPass &sp : sc.passes) {
        PassCost c{sp.kind >= 0, false, 0, 0, 0, 0.0, 1.0};
        if (sp.kind == 6) {
            c.us = 3.8 + 2 * ab * sp.active_amps / 5.4e6;
            c.tabs = (double)sp.tabs.size();
        } else if (c.live) {
            const PassPlan &p = P[sp.first];
            c.d = p.d;
            c.mixes = p.d > 0;
            c.span = span_qubits(p);
            if (p.d >= 4) c.mats = (p.blk.size() * amp_bytes(sc.dt)) << (2 * p.d);
            const double amps = std::ldexp((double)p.blk.size(), sc.n - p.k + p.d);
            const double mem = 2 * ab * amps / 5.4e6, fl = p.d >= 4 ? 8 * amps * (1 << p.d) / (sc.dt == CAST_C128 ? 60e6 : 120e6) : 0;
            const double base = sp.kind == 1 || sp.kind == 2 ? 5.3 : sp.kind == 5 ? 6.5 : p.d >= 5 ? 4.8 : 3.8;
            c.us = base + std::max(mem, fl);
        }
        out.push_back(c);
    }
    return out;
}

// Groups the schedule with tiles of 2^tb amplitudes; *us: predicted time.
std::vector<Span> plan_groups(const Schedule &sc, const std::vector<PassPlan> &P, const std::vector<PassCost> &costs,
                              int tb, double *us) {
    const Tuning &tu = tuning();
    static const double op_us[] = {0.3, 0.7, 0.8, 1.1, 3.0, 5.3}, least_us[] = {0.8, 0.8, 0.8, 0.8, 1.6, 2.6};
    const double tiles = std::ldexp(1.0, sc.n - tb), rounds = std::max(1.0, tiles / 256);
    const double base = tb == 8 && sc.n > 8 ? 8.0 : 5.0;
    double op[6];   // of an operation of dimension d, but for a run's tables
    for (int d = 0; d < 6; ++d) op[d] = op_us[d] * std::ldexp(1.0, tb - 12);
    const double mem = 2 * std::ldexp((double)amp_bytes(sc.dt), sc.n) / 5.2e6;
    const double lone = std::max(mem, 2 * std::ldexp((double)amp_bytes(sc.dt), tb) / 1e5);
    std::vector<Span> out;
    out.reserve(sc.passes.size());
    *us = 0;
    size_t a = 0, mats = 0, live = 0;   // the open group [a, ..): LDS bytes of its dense blocks, passes
    uint64_t need = 0;
    double sep = 0, ops = 0;            // their own launches, and as operations of a tile
    auto close = [&](size_t b) {
        if (a < b) {
            const double grp = base + (tiles <= 256 ? lone + ops : std::max(mem, ops) + 0.3 * std::min(mem, ops));
            if (live > 1 && grp < sep) {
                out.push_back(Span{a, b, need, true});
                *us += grp;
            } else {
                for (size_t i = a; i < b; ++i) out.push_back(Span{i, i + 1, 0, false});
                *us += sep;
            }
        }
        a = b, mats = live = 0, need = 0, sep = ops = 0;
    };
    auto take = [&](const PassCost &c) {
        sep += c.us;
        if (!c.live) return;
        ++live;
        double t = op[std::min(c.d, 5)] * c.tabs;
        if (c.d < 4) t = 0.1 + (tiles <= 256 ? 1.2 * t : t);
        else t = std::max(t, 0.55 * op_us[std::min(c.d, 5)]) * (sc.dt == CAST_C64 ? 0.52 : 1.0);
        ops += std::max(least_us[std::min(c.d, 5)], t * rounds);
    };
    for (size_t i = 0; i < sc.passes.size(); ++i) {
        const PassCost &c = costs[i];
        if (!c.mixes) {
            take(c);
            continue;
        }
        const PassPlan &p = P[sc.passes[i].first];
        int w = 0;
        bool fits = p.d <= kGroupMaxD && window_of(c.span, tb, &w);
        // sixteen columns on tile bits that are no targets; and the knobs keep
        // a block off the matrix cores, or to three products, in single passes
        if (fits && p.d >= 4)
            fits = tb - p.k >= 4 && c.mats <= kBlkMatBytes && p.d >= tu.mfma_min_d[sc.dt] && p.d < tu.mfma_3m_min_d[sc.dt];
        if (!fits) {
            close(i);
            out.push_back(Span{i, i + 1, 0, false});
            *us += c.us;
            a = i + 1;
            continue;
        }
        if (!window_of(need | c.span, tb, &w) || mats + c.mats > kBlkMatBytes) close(i);
        need |= c.span;
        mats += c.mats;
        take(c);
    }
    close(sc.passes.size());
    return out;
}

}  // namespace

cast_status tile_groups(cast_fused *f, const Schedule &sc, cast_dtype dt, bool upload, BlockedPlan **out) {
    BlockedPlan *&bp = f->groups[dt];
    // (an environment variable for both dtypes may ask for more than this one's tile)
    const int most = 31 - __builtin_clz(kBlkTileBytes / (uint32_t)amp_bytes(dt));
    const int knob = std::min(tuning().blocked_tile_bits[dt], most);
    const int mfma = tuning().mfma_min_d[dt], m3 = tuning().mfma_3m_min_d[dt];
    if (bp && (bp->knob_tb != knob || bp->knob_mfma != mfma || bp->knob_3m != m3 ||
               bp->nt != blocked_threads(dt, bp->tb))) {
        blocked_free(bp);
        bp = nullptr;
    }
    if (!bp) {
        const std::vector<PassPlan> &P = f->plans;
        const std::vector<PassCost> costs = pass_costs(sc, P);
        std::vector<Span> best;
        int best_tb = 0;
        double best_us = 0;
        for (int tb = std::min(8, std::min(knob, sc.n)); tb <= std::min(knob, sc.n); ++tb) {
            if (tb < 8) continue;   // 256 threads, one amplitude each
            double us;
            std::vector<Span> g = plan_groups(sc, P, costs, tb, &us);
            if (!best_tb || us <= best_us) best = std::move(g), best_tb = tb, best_us = us;
        }
        auto *p = new BlockedPlan;
        p->tb = best_tb;
        p->knob_tb = knob, p->knob_mfma = mfma, p->knob_3m = m3;
        p->nt = blocked_threads(dt, best_tb);
        if (!best_tb)
            for (size_t i = 0; i < sc.passes.size(); ++i) best.push_back(Span{i, i + 1, 0, false});
        const std::vector<size_t> off = plan_offsets(P, dt);
        p->passes.reserve(best.size());
        p->gates.reserve(P.size() + 16);
        p->ent.reserve(16 * P.size());
        for (const Span &g : best) {
            if (!g.group) {
                BlockedPlan::Pass ps;
                ps.first = sc.passes[g.a].first, ps.count = sc.passes[g.a].count, ps.gate = g.a;
                p->passes.push_back(ps);
                continue;
            }
            const size_t first = sc.passes[g.a].first, end = sc.passes[g.b - 1].first + sc.passes[g.b - 1].count;
            std::vector<size_t> cur;
            for (size_t i = first; i < end; ++i)
                if (!P[i].identity()) cur.push_back(i);
            emit_segment(p, P, off, sc.n, dt, cur, first, end - first, g.need);
        }
        bp = p;
    }
    if (upload)
        if (cast_status rc = upload_tables(f, bp, dt)) return rc;
    *out = bp;
    return CAST_OK;
}

bool groups_ready(const cast_fused *f, const BlockedPlan &bp, cast_dtype dt) {
    return f->dev[dt].ptr && (bp.dev || bp.gates.empty());
}

size_t group_count(const BlockedPlan &bp) { return bp.passes.size(); }

GroupInfo group_info(const BlockedPlan &bp, size_t i) {
    const BlockedPlan::Pass &ps = bp.passes[i];
    return GroupInfo{ps.first, ps.count, ps.segment ? ps.seg.tb : 0, ps.segment ? ps.seg.nt : 0};
}

cast_status launch_group(cast_sv *sv, const cast_fused *f, const BlockedPlan &bp, size_t i, size_t *pass) {
    const BlockedPlan::Pass &ps = bp.passes[i];
    *pass = ps.gate;
    if (!ps.segment) return CAST_OK;
    *pass = (size_t)-1;
    return launch_segment(sv, f, bp, ps.seg);
}

}  // namespace cast

using namespace cast;

extern "C" {

cast_status apply_circuit_blocked(cast_sv *sv, const cast_fused *f) {
    if (cast_status rc = check(sv)) return rc;
    BlockedPlan *bp;
    if (cast_status rc = prepare(f, sv->n, sv->dt, true, &bp)) return rc;
    for (size_t i = 0; i < bp->passes.size(); ++i)
        if (cast_status rc = launch(sv, f, *bp, i)) return rc;
    return CAST_OK;
}

cast_status apply_circuit_blocked_timed(cast_sv *sv, const cast_fused *f, float *pass_ms) {
    if (cast_status rc = check(sv)) return rc;
    if (!pass_ms) return fail(CAST_EINVAL, "NULL argument");
    BlockedPlan *bp;
    if (cast_status rc = prepare(f, sv->n, sv->dt, true, &bp)) return rc;
    const size_t np = bp->passes.size();
    std::vector<hipEvent_t> ev(np + 1, nullptr);
    cast_status rc = CAST_OK;
    for (auto &e : ev)
        if (hipEventCreate(&e) != hipSuccess) rc = fail(CAST_EHIP, "hipEventCreate failed");
    if (!rc && hipEventRecord(ev[0], sv->stream) != hipSuccess) rc = fail(CAST_EHIP, "hipEventRecord failed");
    for (size_t i = 0; i < np && !rc; ++i) {
        rc = launch(sv, f, *bp, i);
        if (!rc && hipEventRecord(ev[i + 1], sv->stream) != hipSuccess) rc = fail(CAST_EHIP, "hipEventRecord failed");
    }
    if (!rc && hipEventSynchronize(ev[np]) != hipSuccess) rc = fail(CAST_EHIP, "hipEventSynchronize failed");
    for (size_t i = 0; i < np && !rc; ++i)
        if (hipEventElapsedTime(&pass_ms[i], ev[i], ev[i + 1]) != hipSuccess)
            rc = fail(CAST_EHIP, "hipEventElapsedTime failed");
    for (auto &e : ev)
        if (e) (void)hipEventDestroy(e);
    return rc;
}

cast_status blocked_info(const cast_fused *f, int n, cast_dtype dt, size_t *n_passes) {
    if (!n_passes) return fail(CAST_EINVAL, "NULL argument");
    BlockedPlan *bp;
    if (cast_status rc = prepare(f, n, dt, false, &bp)) return rc;
    *n_passes = bp->passes.size();
    return CAST_OK;
}

cast_status blocked_pass_info(const cast_fused *f, int n, cast_dtype dt, size_t i, size_t *first, size_t *count,
                              int *tile_bits, int *window, int *high_qubits) {
    BlockedPlan *bp;
    if (cast_status rc = prepare(f, n, dt, false, &bp)) return rc;
    if (i >= bp->passes.size()) return fail(CAST_EINVAL, "pass index out of range");
    const BlockedPlan::Pass &ps = bp->passes[i];
    if (first) *first = ps.first;
    if (count) *count = ps.count;
    if (tile_bits) *tile_bits = ps.segment ? ps.seg.tb : 0;
    if (window) *window = ps.segment ? ps.seg.w : 0;
    if (high_qubits) {
        for (int j = 0; j < kBlkMaxHigh; ++j) high_qubits[j] = -1;
        if (ps.segment)
            for (int j = 0; j < ps.seg.nh; ++j) high_qubits[j] = ps.seg.qh[j];
    }
    return CAST_OK;
}

}  // extern "C"
