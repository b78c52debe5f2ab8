// pdmi_layout.cpp -- family search, node renumbering and the device layout (sliced
// and staged) of new problems.
#include "pdmi_host.h"

namespace pdmi {
namespace host {

// ------------------------------------------------------------------ family search

// Family of every node (Eq. family, self excluded): bin nodes into cubic cells slightly
// wider than delta, test the 27 surrounding cells, sort each row ascending.
void family_search(int64_t n, const double* x, double delta, std::vector<int64_t>& row_ptr,
                   std::vector<int32_t>& col)
{
    double lo[3], hi[3];
    for (int d = 0; d < 3; ++d) lo[d] = hi[d] = x[d];
    for (int64_t i = 1; i < n; ++i)
        for (int d = 0; d < 3; ++d) {
            lo[d] = std::min(lo[d], x[3 * i + d]);
            hi[d] = std::max(hi[d], x[3 * i + d]);
        }
    const double h = delta * (1.0 + 1e-9);
    int64_t dim[3];
    for (int d = 0; d < 3; ++d) {
        const double span = (hi[d] - lo[d]) / h;
        if (!(span < 4.0e6)) fail(PD_ERANGE, "domain spans too many horizon cells");
        dim[d] = static_cast<int64_t>(std::floor(span)) + 1;
    }
    const int64_t ncell = dim[0] * dim[1] * dim[2];
    if (ncell > (int64_t(1) << 31)) fail(PD_ERANGE, "too many cells for the family search");
    auto cell_of = [&](int64_t i, int64_t* c3) {
        for (int d = 0; d < 3; ++d) {
            int64_t c = static_cast<int64_t>(std::floor((x[3 * i + d] - lo[d]) / h));
            c3[d] = std::min(std::max<int64_t>(c, 0), dim[d] - 1);
        }
    };
    std::vector<int64_t> cstart(ncell + 1, 0), items(n);
    std::vector<int64_t> cid(n);
    for (int64_t i = 0; i < n; ++i) {
        int64_t c3[3];
        cell_of(i, c3);
        cid[i] = (c3[2] * dim[1] + c3[1]) * dim[0] + c3[0];
        ++cstart[cid[i] + 1];
    }
    for (int64_t c = 0; c < ncell; ++c) cstart[c + 1] += cstart[c];
    {
        std::vector<int64_t> fill(cstart.begin(), cstart.end() - 1);
        for (int64_t i = 0; i < n; ++i) items[fill[cid[i]]++] = i;
    }
    const double d2max = delta * delta;
    std::vector<int64_t> count(n, 0);
    std::atomic<bool> coincident{false};  // a zero-length bond has no stretch
    // pass 1: counts; pass 2: fill and sort
    for (int pass = 0; pass < 2; ++pass) {
        if (pass == 1) {
            row_ptr.assign(n + 1, 0);
            for (int64_t i = 0; i < n; ++i) row_ptr[i + 1] = row_ptr[i] + count[i];
            if (row_ptr[n] > std::numeric_limits<int32_t>::max())
                fail(PD_ERANGE, "family has 2^31 or more slots");
            col.assign(static_cast<size_t>(row_ptr[n]), 0);
        }
        parallel_for(n, [&](int64_t i0, int64_t i1) {
            for (int64_t i = i0; i < i1; ++i) {
                int64_t c3[3];
                cell_of(i, c3);
                int64_t w = pass ? row_ptr[i] : 0;
                for (int64_t z = std::max<int64_t>(c3[2] - 1, 0); z <= std::min(c3[2] + 1, dim[2] - 1); ++z)
                    for (int64_t y = std::max<int64_t>(c3[1] - 1, 0); y <= std::min(c3[1] + 1, dim[1] - 1); ++y)
                        for (int64_t xx = std::max<int64_t>(c3[0] - 1, 0); xx <= std::min(c3[0] + 1, dim[0] - 1);
                             ++xx) {
                            const int64_t c = (z * dim[1] + y) * dim[0] + xx;
                            for (int64_t p = cstart[c]; p < cstart[c + 1]; ++p) {
                                const int64_t j = items[p];
                                if (j == i) continue;
                                const double a = x[3 * j + 0] - x[3 * i + 0];
                                const double b = x[3 * j + 1] - x[3 * i + 1];
                                const double e = x[3 * j + 2] - x[3 * i + 2];
                                double d2 = a * a + b * b;
                                d2 = d2 + e * e;
                                if (!(d2 <= d2max)) continue;
                                if (d2 == 0.0) coincident = true;
                                if (pass) col[w] = static_cast<int32_t>(j);
                                ++w;
                            }
                        }
                if (pass)
                    std::sort(col.begin() + row_ptr[i], col.begin() + w);
                else
                    count[i] = w;
            }
        });
        if (coincident) fail(PD_EINVAL, "two nodes share a position (a zero-length bond has no stretch)");
    }
}

// ------------------------------------------------------------------ device layout

// Spacing estimate: the smallest bond length among the first rows.
static double spacing_estimate(const Inst& I)
{
    double best = std::numeric_limits<double>::infinity();
    const int64_t rows = std::min<int64_t>(I.n, 4096);
    for (int64_t i = 0; i < rows; ++i)
        for (int64_t b = I.row_ptr[i]; b < I.row_ptr[i + 1]; ++b) {
            const int64_t j = I.col[b];
            double s = 0.0;
            for (int d = 0; d < 3; ++d) {
                const double t = I.x[3 * j + d] - I.x[3 * i + d];
                s += t * t;
            }
            best = std::min(best, std::sqrt(s));
        }
    if (!(best > 0.0) || !std::isfinite(best)) best = I.horizon > 0 ? I.horizon : 1.0;
    return best;
}

static uint64_t spread3(uint64_t v)
{
    v &= 0x1fffff;
    v = (v | v << 32) & 0x1f00000000ffffULL;
    v = (v | v << 16) & 0x1f0000ff0000ffULL;
    v = (v | v << 8) & 0x100f00f00f00f00fULL;
    v = (v | v << 4) & 0x10c30c30c30c30c3ULL;
    v = (v | v << 2) & 0x1249249249249249ULL;
    return v;
}

// Device-local node order of one instance.
static void node_order(Inst& I, int order, double h)
{
    I.iperm.assign(I.n, 0);
    std::vector<int64_t> p(I.n);
    std::iota(p.begin(), p.end(), 0);
    if (order == PD_ORDER_MORTON && I.n > 1) {
        double lo[3];
        for (int d = 0; d < 3; ++d) lo[d] = I.x[d];
        for (int64_t i = 1; i < I.n; ++i)
            for (int d = 0; d < 3; ++d) lo[d] = std::min(lo[d], I.x[3 * i + d]);
        std::vector<uint64_t> key(I.n);
        for (int64_t i = 0; i < I.n; ++i) {
            uint64_t k = 0;
            for (int d = 0; d < 3; ++d) {
                double q = std::floor((I.x[3 * i + d] - lo[d]) / h + 0.5);
                q = std::min(std::max(q, 0.0), 2097151.0);
                k |= spread3(static_cast<uint64_t>(q)) << d;
            }
            key[i] = k;
        }
        std::stable_sort(p.begin(), p.end(), [&](int64_t a, int64_t b) { return key[a] < key[b]; });
    }
    for (int64_t i = 0; i < I.n; ++i) I.iperm[p[i]] = i;
    I.perm = std::move(p);
}

// Dispatch order of the staged tiles (context-wide indices).  xcd_remap hands each XCD a
// contiguous share of the dispatch positions; within every share the tiles keep their
// device order but those with more slot rows (in buckets of 8) go first, so that the last
// workgroups of a launch are the short ones and the tail of the launch is short.
// Every tile writes only its own nodes, so results do not depend on the order.
static std::vector<int32_t> tile_dispatch_order(const std::vector<int64_t>& rows)
{
    const int64_t nt = static_cast<int64_t>(rows.size());
    std::vector<int32_t> order(static_cast<size_t>(nt));
    std::iota(order.begin(), order.end(), 0);
    constexpr int64_t X = 8;  // XCDs, as xcd_remap splits the dispatch
    const int64_t m = nt / X, r = nt % X;
    int64_t b0 = 0;
    for (int64_t x = 0; x < X; ++x) {
        const int64_t len = m + (x < r ? 1 : 0);
        std::stable_sort(order.begin() + b0, order.begin() + b0 + len,
                         [&](int32_t a, int32_t b) { return rows[a] / 8 > rows[b] / 8; });
        b0 += len;
    }
    return order;
}

// Order of each row's slots on the device: by the bond offset rounded to the lattice
// spacing (z, then y, then x), so lanes of neighbouring nodes visit neighbours at the
// same relative position together.  On a natural-order lattice this is ascending j.
static std::vector<int32_t> slot_ranks(const Inst& I, double h)
{
    std::vector<int32_t> order(static_cast<size_t>(I.nnz));
    parallel_for(I.n, [&](int64_t i0, int64_t i1) {
        std::vector<std::pair<int64_t, int32_t>> tmp;
        for (int64_t i = i0; i < i1; ++i) {
            const int64_t b0 = I.row_ptr[i], b1 = I.row_ptr[i + 1];
            tmp.clear();
            for (int64_t b = b0; b < b1; ++b) {
                const int64_t j = I.col[b];
                int64_t q[3];
                for (int d = 0; d < 3; ++d)
                    q[d] = static_cast<int64_t>(std::llround((I.x[3 * j + d] - I.x[3 * i + d]) / h));
                const int64_t key = ((q[2] + 4096) * 8192 + (q[1] + 4096)) * 8192 + (q[0] + 4096);
                tmp.emplace_back(key, static_cast<int32_t>(b - b0));
            }
            std::sort(tmp.begin(), tmp.end());
            for (int64_t r = 0; r < b1 - b0; ++r) order[b0 + r] = tmp[r].second;
        }
    });
    return order;
}

// A node and its lattice cell, for the recursive bisection into compact slices.
struct CellNode {
    int32_t q[3];
    int32_t id;
};

// Nodes [lo, hi) into nsl slices of 64 (the last of the instance may be short): cut across
// the longest extent, at a multiple of `group` slices while a part holds more than one
// group, so that the slices of a group are neighbours too.  The cut leaves whole groups of
// about cubic shape on both sides (13 of them across are cut 6 to 7, not in halves: a
// 100 x 25 x 20 lattice stages 4.1 records a node in place of 4.3, 117 x 33 x 33 at horizon 3.14
// 4.5 in place of 4.6).  Nodes of one slice end up in ascending order.
static void bisect(CellNode* p, int64_t lo, int64_t hi, int64_t nsl, int64_t group, int depth)
{
    if (nsl <= 1) {
        std::sort(p + lo, p + hi, [](const CellNode& a, const CellNode& b) { return a.id < b.id; });
        return;
    }
    int32_t mn[3], mx[3];
    for (int d = 0; d < 3; ++d) mn[d] = mx[d] = p[lo].q[d];
    for (int64_t i = lo + 1; i < hi; ++i)
        for (int d = 0; d < 3; ++d) {
            mn[d] = std::min(mn[d], p[i].q[d]);
            mx[d] = std::max(mx[d], p[i].q[d]);
        }
    int ax[3] = {2, 1, 0};  // ties: z first, so that x stays the longest run
    std::stable_sort(ax, ax + 3, [&](int a, int b) { return mx[a] - mn[a] > mx[b] - mn[b]; });
    int64_t left = nsl / 2;
    if (nsl > group) {
        // edge of a cubic group, axes that are thinner than that set aside
        const double T = static_cast<double>(nsl) / static_cast<double>(group);
        double e[3];
        for (int k = 0; k < 3; ++k) e[k] = mx[ax[k]] - mn[ax[k]] + 1;
        double edge = std::cbrt(e[0] * e[1] * e[2] / T);
        if (e[2] < edge) edge = std::sqrt(e[0] * e[1] / T);
        if (e[1] < edge) edge = e[0] / T;
        const double across = std::max(2.0, std::round(e[0] / edge));
        left = std::llround(T * std::floor(0.5 * across) / across) * group;
        left = std::min(std::max(left, group), (nsl - 1) / group * group);
    }
    const int64_t mid = lo + left * kWave;
    std::nth_element(p + lo, p + mid, p + hi, [&](const CellNode& a, const CellNode& b) {
        for (int d : {ax[0], ax[1], ax[2]})
            if (a.q[d] != b.q[d]) return a.q[d] < b.q[d];
        return a.id < b.id;
    });
    std::thread t;
    if (depth > 0 && hi - lo > 8192) {
        try {
            t = std::thread([&] { bisect(p, lo, mid, left, group, depth - 1); });
        } catch (const std::system_error&) {  // no thread to be had: in turn
        }
    }
    if (!t.joinable()) bisect(p, lo, mid, left, group, 0);
    bisect(p, mid, hi, nsl - left, group, depth > 0 ? depth - 1 : 0);  // (throws nothing)
    if (t.joinable()) t.join();
}

// Device-local node order of one instance on the staged layout: compact slices, and within
// a slice lanes by bank class, so that 16 lanes that read the neighbours at one offset
// together find them in different banks.
static void slice_nodes(Inst& I, int64_t group, double h, std::vector<uint8_t>& bank)
{
    double lo[3];
    for (int d = 0; d < 3; ++d) lo[d] = I.x[d];
    for (int64_t i = 1; i < I.n; ++i)
        for (int d = 0; d < 3; ++d) lo[d] = std::min(lo[d], I.x[3 * i + d]);
    std::vector<CellNode> c(static_cast<size_t>(I.n));
    for (int64_t i = 0; i < I.n; ++i) {
        for (int d = 0; d < 3; ++d)
            c[i].q[d] = static_cast<int32_t>(std::min(std::floor((I.x[3 * i + d] - lo[d]) / h + 0.5), 1.0e9));
        c[i].id = static_cast<int32_t>(i);
    }
    // bank class: 48-byte records at indices equal mod 16 share their LDS banks; on a lattice
    // a 4 x 4 patch of nodes covers all 16 classes
    bank.resize(static_cast<size_t>(I.n));
    for (int64_t i = 0; i < I.n; ++i) {
        const auto q = [&](int d) { return static_cast<uint32_t>(c[i].q[d]); };
        bank[i] = static_cast<uint8_t>((q(0) + 12 * q(1) + 3 * q(2)) & 15);
    }
    bisect(c.data(), 0, I.n, (I.n + kWave - 1) / kWave, group, 4);
    I.perm.resize(static_cast<size_t>(I.n));
    I.iperm.resize(static_cast<size_t>(I.n));
    // lanes of a slice: bank class c to lanes c, c + 16, ... as far as they go
    for (int64_t l0 = 0; l0 < I.n; l0 += kWave) {
        const int top = static_cast<int>(std::min<int64_t>(kWave, I.n - l0));
        int next[16];
        int32_t spill[kWave];
        int ns = 0;
        for (int k = 0; k < 16; ++k) next[k] = k;
        for (int l = 0; l < top; ++l) {
            const int32_t id = c[l0 + l].id;
            int& f = next[bank[id]];
            if (f < top) {
                I.perm[l0 + f] = id;
                f += 16;
            } else {
                spill[ns++] = id;
            }
        }
        for (int k = 0, m = 0; m < ns; ++m) {
            while (next[k] >= top) ++k;
            I.perm[l0 + next[k]] = spill[m];
            next[k] += 16;
        }
    }
    for (int64_t l = 0; l < I.n; ++l) I.iperm[I.perm[l]] = l;
}

// Records that fit a workgroup's LDS: beside one other workgroup on the CU, and alone.
struct StageRoom {
    int64_t two, one;
};

// User nodes that the bonds of nsl slices reach, ascending (seen: zeros, and zeros again after).
static void reached(const Inst& I, int64_t slice, int64_t nsl, std::vector<uint8_t>& seen, std::vector<int32_t>& nodes)
{
    nodes.clear();
    for (int64_t l = slice * kWave; l < (slice + nsl) * kWave; ++l) {
        const int64_t p = I.perm[l];
        if (p < 0) continue;
        for (int64_t b = I.row_ptr[p]; b < I.row_ptr[p + 1]; ++b)
            if (!seen[I.col[b]]) {
                seen[I.col[b]] = 1;
                nodes.push_back(I.col[b]);
            }
    }
    std::sort(nodes.begin(), nodes.end());
    for (int32_t j : nodes) seen[j] = 0;
}

// A tile before it is laid out: its slices and the records it stages.
struct Part {
    int64_t slice = 0, nsl = 0;
    std::vector<int32_t> nodes;  // user nodes reached, ascending
    int32_t nphase = 0, per = 0;
    std::vector<int32_t> at;     // record index of every one in its phase
    std::vector<int32_t> n;      // records per phase
    std::vector<int32_t> pairs;  // per phase and slice of the tile
};

// Two workgroups a CU hide each other's staging, so a part of more than `least` slices whose
// records do not fit a CU's LDS twice is cut in two, and so on.
static void cut_part(const Inst& I, int64_t slice, int64_t nsl, int64_t least, int64_t two, std::vector<uint8_t>& seen,
                     std::vector<Part>& out)
{
    Part p;
    p.slice = slice;
    p.nsl = nsl;
    reached(I, slice, nsl, seen, p.nodes);
    if (nsl > least && static_cast<int64_t>(p.nodes.size()) > two) {
        const int64_t left = (nsl + 1) / 2;
        cut_part(I, slice, left, least, two, seen, out);
        cut_part(I, slice + left, nsl - left, least, two, seen, out);
    } else {
        out.push_back(std::move(p));
    }
}

// Staged layout of one instance: tiles of up to `group` consecutive slices.  The nodes that
// a tile's bonds reach are cut into phases (one unless the families are very large); each
// lane's slots of a phase, in ascending neighbour order, fill its slice's row pairs.  Fills
// the tile, phase and segment tables, dslot_user and ent_idx (index of the slot's record in
// its phase, from 1); returns the slot count.
static int64_t build_staged(Inst& I, int64_t group, const StageRoom& room, const std::vector<uint8_t>& bank)
{
    const int64_t ng = (I.nslices + group - 1) / group;
    std::vector<std::vector<Part>> parts(static_cast<size_t>(ng));
    // Tiles of one slice, if nearly all of them then fit twice and the others do in two phases
    // (1M nodes at horizon 5.015: 785 us a step, two slices a tile and one tile a CU 885), else of two
    // at least, with one tile a CU where they do not fit twice (125000 nodes at 8.015: 450, cut
    // 464).  A problem whose tiles have a CU each has no use for room for two (15625 nodes at 5.015:
    // 20 us in one phase, 23 in two).
    int64_t phase = group > 1 ? room.two : room.one;
    for (int64_t least : {1, 2}) {
        std::atomic<int64_t> tiles{0}, over{0};
        parallel_for(ng, [&](int64_t g0, int64_t g1) {
            std::vector<uint8_t> seen(static_cast<size_t>(I.n), 0);
            for (int64_t g = g0; g < g1; ++g) {
                parts[g].clear();
                cut_part(I, g * group, std::min(group, I.nslices - g * group), least, room.two, seen, parts[g]);
                for (const Part& P : parts[g]) over += static_cast<int64_t>(P.nodes.size()) > room.two;
                tiles += static_cast<int64_t>(parts[g].size());
            }
        }, 64);
        if (over <= tiles / 4) break;
        phase = room.one;
    }
    parallel_for(ng, [&](int64_t g0, int64_t g1) {
        for (int64_t g = g0; g < g1; ++g) {
            for (Part& P : parts[g]) {
                const int64_t R = static_cast<int64_t>(P.nodes.size());
                P.nphase = static_cast<int32_t>((R + phase - 1) / phase);
                P.per = P.nphase ? static_cast<int32_t>((R + P.nphase - 1) / P.nphase) : 0;
                P.at.resize(static_cast<size_t>(R));
                for (int ph = 0; ph < P.nphase; ++ph) {
                    // a record goes to the next place of its bank class (index mod 16); the few that
                    // find their class full take the places left over
                    const int64_t r0 = static_cast<int64_t>(ph) * P.per, r1 = std::min<int64_t>(R, r0 + P.per);
                    const int32_t top = static_cast<int32_t>(r1 - r0);
                    int32_t next[16];
                    for (int c = 0; c < 16; ++c) next[c] = c;
                    for (int64_t r = r0; r < r1; ++r) {
                        int32_t& f = next[bank[P.nodes[r]]];
                        P.at[r] = f < top ? f : -1;
                        if (f < top) f += 16;
                    }
                    int c = 0;
                    for (int64_t r = r0; r < r1; ++r) {
                        if (P.at[r] >= 0) continue;
                        while (next[c] >= top) ++c;
                        P.at[r] = next[c];
                        next[c] += 16;
                    }
                    P.n.push_back(top);
                }
                P.pairs.assign(static_cast<size_t>(P.nphase * P.nsl), 0);
                for (int64_t k = 0; k < P.nsl; ++k)
                    for (int w = 0; w < kWave; ++w) {
                        const int64_t p = I.perm[(P.slice + k) * kWave + w];
                        if (p < 0) continue;
                        const auto last = I.col.begin() + I.row_ptr[p + 1];
                        auto from = I.col.begin() + I.row_ptr[p];
                        for (int ph = 0; ph < P.nphase; ++ph) {
                            const int64_t next = static_cast<int64_t>(ph + 1) * P.per;
                            const auto to = next < R ? std::lower_bound(from, last, P.nodes[next]) : last;
                            int32_t& q = P.pairs[ph * P.nsl + k];
                            q = std::max(q, static_cast<int32_t>((to - from + 1) / 2));
                            from = to;
                        }
                    }
            }
        }
    }, 64);
    I.tiles.clear();
    I.phases.clear();
    I.segs.clear();
    I.tile_rows.clear();
    std::vector<const Part*> part;
    int64_t npair = 0, nlist = 0;
    for (const auto& ps : parts)
        for (const Part& P : ps) {
            part.push_back(&P);
            I.tiles.push_back(TileRec{static_cast<int>(P.slice), static_cast<int>(P.nsl), static_cast<int>(I.phases.size()),
                                      P.nphase, static_cast<int>(nlist), P.nphase ? P.n[0] : 0, 0,
                                      static_cast<int>(I.segs.size())});
            int64_t total = 0;
            for (int ph = 0; ph < P.nphase; ++ph) {
                I.phases.push_back(int2{static_cast<int>(nlist), P.n[ph]});
                nlist += P.n[ph];
                for (int64_t k = 0; k < P.nsl; ++k) {
                    const int32_t q = P.pairs[ph * P.nsl + k];
                    I.segs.push_back(int2{static_cast<int>(npair), q});
                    npair += q;
                    total += 2 * q;
                }
            }
            I.tile_rows.push_back(total);
        }
    if (npair * 2 * kWave >= std::numeric_limits<int32_t>::max())
        fail(PD_ERANGE, "device problem needs 2^31 or more slots");
    I.list.resize(static_cast<size_t>(nlist));
    I.dslot_user.resize(static_cast<size_t>(npair * 2 * kWave));
    I.ent_idx.resize(static_cast<size_t>(npair * 2 * kWave));
    parallel_for(static_cast<int64_t>(part.size()), [&](int64_t t0, int64_t t1) {
        std::vector<int32_t> at(static_cast<size_t>(I.n), 0);  // index of a node in the tile's list
        for (int64_t t = t0; t < t1; ++t) {
            const Part& P = *part[t];
            const TileRec& T = I.tiles[t];
            const int64_t R = static_cast<int64_t>(P.nodes.size());
            for (int64_t r = 0; r < R; ++r) at[P.nodes[r]] = P.at[r];
            for (int ph = 0; ph < P.nphase; ++ph) {
                const int2 S = I.phases[T.phase + ph];
                const int64_t r0 = static_cast<int64_t>(ph) * P.per, r1 = std::min<int64_t>(R, r0 + P.per);
                for (int64_t r = r0; r < r1; ++r)
                    I.list[S.x + P.at[r]] = static_cast<int32_t>(I.node_off + I.iperm[P.nodes[r]]);
                for (int k = 0; k < T.nslices; ++k) {
                    const int2 g = I.segs[T.seg + ph * T.nslices + k];
                    for (int w = 0; w < kWave; ++w) {
                        const int64_t p = I.perm[(static_cast<int64_t>(T.slice) + k) * kWave + w];
                        int64_t b = 0, b1 = 0;
                        if (p >= 0) {
                            b = I.row_ptr[p];
                            b1 = I.row_ptr[p + 1];
                            const auto first = I.col.begin() + b, last = I.col.begin() + b1;
                            if (ph > 0) b += std::lower_bound(first, last, P.nodes[r0]) - first;
                            if (r1 < R) b1 = std::lower_bound(first, last, P.nodes[r1]) - I.col.begin();
                        }
                        for (int64_t q = 0; q < 2 * static_cast<int64_t>(g.y); ++q) {
                            const int64_t ds = (g.x + q / 2) * (2 * kWave) + 2 * w + (q & 1);
                            const bool real = b + q < b1;
                            I.dslot_user[ds] = real ? static_cast<int32_t>(b + q) : -1;
                            I.ent_idx[ds] = real ? static_cast<uint16_t>(at[I.col[b + q]] + 1) : 0;
                        }
                    }
                }
            }
        }
    }, 64);
    return npair * 2 * kWave;
}

// Records a phase may hold: what fits a workgroup's LDS in every kernel that the problem can
// run with what it carries now (48 bytes a record, 8 for a weight of its node, 16 for the
// state-based pair, 24 for the adjoint velocity).
static StageRoom stage_room(const pd_ctx* ctx)
{
    bool vol = false, knode = false, corr = false, osb = false;
    for (const Inst& I : ctx->inst) {
        vol |= !I.vols.empty();
        knode |= !I.knode.empty();
        corr |= I.has_corr;
        osb |= I.osb;
    }
    const int64_t weight = vol || knode || corr ? 8 : 0;
    int64_t per = 48 + weight;
    if (osb) per = 64 + weight;
    if (ctx->adjoint) per = std::max<int64_t>(per, 72 + (vol ? 8 : 0) + (knode ? 8 : 0));
    const int64_t fixed = 1280;  // the step kernel's lists of slots to settle (1 KB), in the hardware's steps
    return StageRoom{(kLdsBytes / 2 - fixed) / per - 1, std::min<int64_t>((kLdsBytes - fixed) / per - 1, kEntIdx)};
}

// Slices of a tile, from the slices of all instances: large tiles stage each record for more
// bonds, but a launch wants about two a CU.  us/step with 4, 2, 1 slices a tile: 1M nodes
// (15625 slices) 194, 220, 291; 262144 nodes 52.9, 56.0, 69.5; 125000 nodes 36.0, 37.1, 41.7; 50000
// nodes 17.6, 17.2, 18.6; 1000 nodes 16.1, 10.6, 8.1.  Damage laws follow the same rule (1M nodes,
// nothing softened: 204, 227, 307; 127k nodes with a grown crack, 2 and 1: 39.1, 45.0).  The
// mapping's lanes have no say in it.
static int64_t tile_slices(const pd_ctx* ctx)
{
    int64_t nsl = 0;
    for (const Inst& I : ctx->inst) nsl += (I.n + kWave - 1) / kWave;
    return nsl >= 3072 ? kTileSlices : nsl >= 512 ? 2 : 1;
}

static void check_nodes(int64_t nn)
{
    if (nn >= std::numeric_limits<int32_t>::max()) fail(PD_ERANGE, "device problem needs 2^31 or more nodes or slots");
    if (nn + 1 >= (int64_t(1) << 24))
        fail(PD_ERANGE, "device problem needs 2^24 or more node records (the gather uses 24-bit indices)");
}

// After a change of what the kernels stage: a phase that no longer fits (twice, where it did) is
// cut anew, and so are tiles that were cut for want of room there is now.  Done by the next call
// that runs a kernel.
void fit_stage(pd_ctx* ctx)
{
    if (!ctx->laid || ctx->mapping != PD_MAP_STAGED) return;
    const StageRoom r = stage_room(ctx);
    ctx->recut = (r.two < ctx->stage_two && ctx->stage_max > r.two) || (r.two > ctx->stage_two && ctx->stage_cut);
}

// Called by every entry point that needs the device problem: the device, and the problem on it.
void laid_out(pd_ctx* ctx)
{
    set_device(ctx);
    if (ctx->built && !ctx->laid) build_layout(ctx);
}

// The same for those that run its kernels: with tiles for what the problem holds now.  The state
// is kept, break steps and the acceleration's validity included.
void ready(pd_ctx* ctx)
{
    laid_out(ctx);
    if (!ctx->recut) return;
    auto S = std::make_shared<HostState>(snapshot(ctx));
    for (const Inst& I : ctx->inst) S->bstep.push_back(bstep_of(ctx, I));
    ctx->kept = std::move(S);
    build_layout(ctx);
}

// Allocate and fill the device problem for ctx->lanes from the instances' user data and the
// kept state.
void build_layout(pd_ctx* ctx)
{
    const HostState* const S = ctx->kept.get();
    ctx->laid = false;
    const bool staged = ctx->mapping == PD_MAP_STAGED;
    const int G = staged ? 1 : ctx->lanes, W = kWave / G;
    ctx->drop_graphs();
    ctx->tape_valid = false;
    ctx->ck.release();
    ctx->kslot.release();  // slot layout changes: re-uploaded in full below
    int64_t nn = 0, nsl = 0, ns = 0;
    std::vector<int64_t> sp;
    std::vector<int32_t> sT, sI, list;
    std::vector<TileRec> tiles;
    std::vector<int2> phases, segs;
    std::vector<int64_t> tile_rows;
    int64_t stage_max = 0;
    const StageRoom room = stage_room(ctx);
    const int64_t group = tile_slices(ctx);
    ctx->stage_two = room.two;
    ctx->stage_cut = false;
    for (size_t ii = 0; ii < ctx->inst.size(); ++ii) {
        Inst& I = ctx->inst[ii];
        const double h = spacing_estimate(I);
        std::vector<uint8_t> bank;
        if (staged)
            slice_nodes(I, group, h, bank);
        else
            node_order(I, ctx->order, h);
        I.n_pad = (I.n + W - 1) / W * W;
        I.perm.resize(static_cast<size_t>(I.n_pad), -1);
        I.node_off = nn;
        I.nslices = I.n_pad / W;
        I.slice_off = nsl;
        I.dslot_off = ns;
        std::vector<int64_t> T(static_cast<size_t>(I.nslices), 0);
        std::vector<int64_t> start(static_cast<size_t>(I.nslices));
        int64_t nds = 0;
        if (ctx->mapping == PD_MAP_STAGED) {
            nds = build_staged(I, group, room, bank);
            ctx->stage_cut |= static_cast<int64_t>(I.tiles.size()) > (I.nslices + group - 1) / group || I.phases.size() > I.tiles.size();
            if (ns + nds >= std::numeric_limits<int32_t>::max())
                fail(PD_ERANGE, "device problem needs 2^31 or more nodes or slots");
            for (TileRec t : I.tiles) {
                t.slice += static_cast<int>(nsl);
                t.phase += static_cast<int>(phases.size());
                t.list += static_cast<int>(list.size());
                t.seg += static_cast<int>(segs.size());
                t.inst = static_cast<int>(ii);
                tiles.push_back(t);
            }
            for (int2 g : I.segs) segs.push_back(int2{g.x + static_cast<int>(ns / (2 * kWave)), g.y});
            for (int2 p : I.phases) {
                phases.push_back(int2{p.x + static_cast<int>(list.size()), p.y});
                stage_max = std::max<int64_t>(stage_max, p.y);
            }
            list.insert(list.end(), I.list.begin(), I.list.end());
            tile_rows.insert(tile_rows.end(), I.tile_rows.begin(), I.tile_rows.end());
        } else {
            const std::vector<int32_t> ranks = slot_ranks(I, h);
            // slice row counts
            for (int64_t s = 0; s < I.nslices; ++s)
                for (int w = 0; w < W; ++w) {
                    const int64_t p = I.perm[s * W + w];
                    if (p >= 0) T[s] = std::max<int64_t>(T[s], (I.row_ptr[p + 1] - I.row_ptr[p] + G - 1) / G);
                }
            for (auto& t : T) t = (t + kRowUnroll - 1) / kRowUnroll * kRowUnroll;
            for (int64_t s = 0; s < I.nslices; ++s) {
                start[s] = nds;
                nds += T[s] * kWave;
            }
            I.dslot_user.assign(static_cast<size_t>(nds), -1);
            parallel_for(I.nslices, [&](int64_t s0, int64_t s1) {
                for (int64_t s = s0; s < s1; ++s)
                    for (int w = 0; w < W; ++w) {
                        const int64_t p = I.perm[s * W + w];
                        if (p < 0) continue;
                        const int64_t b0 = I.row_ptr[p], len = I.row_ptr[p + 1] - b0;
                        for (int64_t r = 0; r < len; ++r) {
                            const int64_t t = r / G, g = r % G;
                            I.dslot_user[start[s] + t * kWave + w * G + g] = static_cast<int32_t>(b0 + ranks[b0 + r]);
                        }
                    }
            });
        }
        I.n_dslots = nds;
        I.s_start = start;
        I.s_T = T;
        for (int64_t s = 0; s < I.nslices; ++s) {
            sp.push_back(ns + start[s]);
            if (T[s] > std::numeric_limits<int32_t>::max()) fail(PD_ERANGE, "row too long");
            sT.push_back(static_cast<int32_t>(T[s]));
            sI.push_back(static_cast<int32_t>(ii));
        }
        nn += I.n_pad;
        nsl += I.nslices;
        ns += nds;
    }
    if (ns >= std::numeric_limits<int32_t>::max()) fail(PD_ERANGE, "device problem needs 2^31 or more nodes or slots");
    check_nodes(nn);
    ctx->nn = nn;
    ctx->nslices = nsl;
    ctx->ns = ns;
    for (int b = 0; b < 2; ++b) {
        ctx->rec[b].alloc(rec_bytes(nn));
        if (fp32(ctx))
            ctx->um[b].alloc(static_cast<size_t>(3 * nn) * sizeof(double));
        else
            ctx->um[b].release();
    }
    ctx->v.alloc(static_cast<size_t>(3 * nn) * sizeof(double));
    ctx->a.alloc(static_cast<size_t>(3 * nn) * sizeof(double));
    const size_t spare = kSpareRows * kWave;
    ctx->bstep.alloc((static_cast<size_t>(ns) + spare) * sizeof(int32_t));
    if (ctx->mapping == PD_MAP_STAGED) {
        ctx->col.release();
        ctx->ent.alloc((static_cast<size_t>(ns) + spare) * sizeof(uint16_t));
    } else {
        ctx->ent.release();
        ctx->col.alloc((static_cast<size_t>(ns) + spare) * sizeof(int32_t));
    }
    ctx->slice_ptr.alloc(sp.size() * sizeof(int64_t));
    ctx->slice_T.alloc(sT.size() * sizeof(int32_t));
    ctx->slice_inst.alloc(sI.size() * sizeof(int32_t));
    ctx->ntiles = static_cast<int64_t>(tiles.size());
    ctx->stage_max = stage_max;
    if (staged) {
        ctx->tiles.alloc(tiles.size() * sizeof(TileRec));
        ctx->phases.alloc(phases.size() * sizeof(int2));
        ctx->segs.alloc(segs.size() * sizeof(int2));
        ctx->list.alloc(list.size() * sizeof(int32_t));
    } else {
        for (DevBuf* d : {&ctx->tiles, &ctx->phases, &ctx->segs, &ctx->list}) d->release();
    }
    ctx->params.alloc(ctx->inst.size() * sizeof(InstParams));
    ctx->bc_id.alloc(static_cast<size_t>(nn) * sizeof(int32_t));
    ctx->step_base.alloc(sizeof(int64_t));
    ctx->status.alloc(sizeof(int32_t));
    ctx->phi.alloc(static_cast<size_t>(nn) * sizeof(double));
    hip_check(hipMemsetAsync(ctx->rec[0].p, 0, ctx->rec[0].bytes, ctx->stream), "hipMemsetAsync");
    hip_check(hipMemsetAsync(ctx->rec[1].p, 0, ctx->rec[1].bytes, ctx->stream), "hipMemsetAsync");
    hip_check(hipMemsetAsync(ctx->v.p, 0, ctx->v.bytes, ctx->stream), "hipMemsetAsync");
    for (int b = 0; b < 2; ++b)
        if (ctx->um[b].p) hip_check(hipMemsetAsync(ctx->um[b].p, 0, ctx->um[b].bytes, ctx->stream), "hipMemsetAsync");
    hip_check(hipMemsetAsync(ctx->a.p, 0, ctx->a.bytes, ctx->stream), "hipMemsetAsync");
    const int32_t status = S ? S->status : 0;
    upload(ctx->status, &status, sizeof status, 0, ctx->stream);
    if (ctx->col.p) hip_check(hipMemsetAsync(ctx->col.p, 0, ctx->col.bytes, ctx->stream), "hipMemsetAsync");
    if (ctx->ent.p) hip_check(hipMemsetAsync(ctx->ent.p, 0, ctx->ent.bytes, ctx->stream), "hipMemsetAsync");
    upload(ctx->slice_ptr, sp.data(), sp.size() * sizeof(int64_t), 0, ctx->stream);
    upload(ctx->slice_T, sT.data(), sT.size() * sizeof(int32_t), 0, ctx->stream);
    upload(ctx->slice_inst, sI.data(), sI.size() * sizeof(int32_t), 0, ctx->stream);
    if (ctx->mapping == PD_MAP_STAGED) {
        std::vector<TileRec> sorted;
        sorted.reserve(tiles.size());
        for (int32_t t : tile_dispatch_order(tile_rows)) sorted.push_back(tiles[t]);
        upload(ctx->tiles, sorted.data(), sorted.size() * sizeof(TileRec), 0, ctx->stream);
        upload(ctx->phases, phases.data(), phases.size() * sizeof(int2), 0, ctx->stream);
        upload(ctx->segs, segs.data(), segs.size() * sizeof(int2), 0, ctx->stream);
        upload(ctx->list, list.data(), list.size() * sizeof(int32_t), 0, ctx->stream);
    }
    const int64_t st = ctx->step;
    upload(ctx->step_base, &st, sizeof st, 0, ctx->stream);
    const double sentinel[6] = {1e10, 1e10, 1e10, 0.0, 0.0, 0.0};
    for (int b = 0; b < 2; ++b) upload(ctx->rec[b], sentinel, sizeof sentinel, static_cast<size_t>(nn) * 48, ctx->stream);
    sync(ctx);
    struct Unfinished {  // (the uploads below need the flag)
        pd_ctx* ctx;
        ~Unfinished()
        {
            if (ctx) ctx->laid = false;
        }
    } unfinished{ctx};
    ctx->laid = true;
    upload_params(ctx);
    upload_bcs(ctx);
    upload_stiffness(ctx);
    upload_volumes(ctx);
    upload_node_weights(ctx);
    upload_body(ctx);
    upload_laws(ctx);
    upload_osb(ctx);
    for (size_t ii = 0; ii < ctx->inst.size(); ++ii) {
        Inst& I = ctx->inst[ii];
        std::vector<double> zeros(static_cast<size_t>(3 * I.n), 0.0);
        upload_state(ctx, I, S ? S->u[ii].data() : zeros.data(), S ? S->v[ii].data() : nullptr,
                     S ? S->a[ii].data() : nullptr);
        const double* sm = (S && !S->smax[ii].empty()) ? S->smax[ii].data() : nullptr;
        upload_col(ctx, I, S ? S->broken[ii].data() : nullptr, false, sm);
        if (S && !S->bstep.empty()) upload_bstep(ctx, I, S->bstep[ii].data());
    }
    {  // device node of every user node, for readouts into device memory
        std::vector<int64_t> dn;
        for (auto& I : ctx->inst) {
            I.user_off = static_cast<int64_t>(dn.size());
            for (int64_t u = 0; u < I.n; ++u) dn.push_back(I.node_off + I.iperm[u]);
        }
        ctx->unode.alloc(dn.size() * sizeof(int64_t));
        upload(ctx->unode, dn.data(), dn.size() * sizeof(int64_t), 0, ctx->stream);
    }
    ctx->cur = 0;
    ctx->vv_ahead = false;
    ctx->recut = false;
    ctx->kept.reset();
    unfinished.ctx = nullptr;
}

void validate_coords(int64_t n, const double* coords, double horizon)
{
    if (n < 1) fail(PD_EINVAL, "n must be >= 1");
    if (n >= std::numeric_limits<int32_t>::max()) fail(PD_ERANGE, "n must be < 2^31 - 1");
    if (!coords) fail(PD_EINVAL, "coords is NULL");
    if (!(horizon > 0.0) || !std::isfinite(horizon)) fail(PD_EINVAL, "horizon must be positive and finite");
    for (int64_t i = 0; i < 3 * n; ++i)
        if (!std::isfinite(coords[i])) fail(PD_EINVAL, "coords must be finite");
}

// A caller's family (pd_set_family): CSR with rows strictly ascending, no self bonds,
// every bond present in both directions, no zero-length bond.  Returns the longest bond.
double validate_family(int64_t n, const double* x, const int64_t* row_ptr, const int32_t* col)
{
    if (!row_ptr || row_ptr[0] != 0) fail(PD_EINVAL, "row_ptr must start at 0");
    for (int64_t i = 0; i < n; ++i)
        if (row_ptr[i + 1] < row_ptr[i]) fail(PD_EINVAL, "row_ptr must be non-decreasing");
    if (row_ptr[n] >= std::numeric_limits<int32_t>::max()) fail(PD_ERANGE, "family has 2^31 or more slots");
    if (row_ptr[n] > 0 && !col) fail(PD_EINVAL, "col is NULL");
    std::atomic<int> bad{0};
    std::vector<double> longest(static_cast<size_t>(n), 0.0);
    parallel_for(n, [&](int64_t i0, int64_t i1) {
        for (int64_t i = i0; i < i1; ++i)
            for (int64_t b = row_ptr[i]; b < row_ptr[i + 1]; ++b) {
                const int64_t j = col[b];
                if (j < 0 || j >= n || j == i) { bad = 1; return; }
                if (b > row_ptr[i] && col[b - 1] >= col[b]) { bad = 2; return; }
                if (!std::binary_search(col + row_ptr[j], col + row_ptr[j + 1], static_cast<int32_t>(i))) {
                    bad = 3;
                    return;
                }
                double L2 = 0.0;
                for (int d = 0; d < 3; ++d) L2 += (x[3 * j + d] - x[3 * i + d]) * (x[3 * j + d] - x[3 * i + d]);
                if (!(L2 > 0.0)) { bad = 4; return; }
                longest[i] = std::max(longest[i], std::sqrt(L2));
            }
    });
    switch (bad.load()) {
    case 1: fail(PD_EINVAL, "family: neighbour id out of range or a self bond");
    case 2: fail(PD_EINVAL, "family: rows must be strictly ascending");
    case 3: fail(PD_EINVAL, "family: every bond must appear in both directions");
    case 4: fail(PD_EINVAL, "family: zero-length bond (coincident nodes)");
    default: break;
    }
    double h = 0.0;
    for (double v : longest) h = std::max(h, v);
    return h > 0.0 ? h : 1.0;
}

void new_problem(pd_ctx* ctx, int32_t ninst, const int64_t* n, const double* const* coords, const double* horizon,
                 int order, const int64_t* user_row_ptr, const int32_t* user_col)
{
    if (order != PD_ORDER_NATURAL && order != PD_ORDER_MORTON && order != PD_ORDER_AUTO)
        fail(PD_EINVAL, "unknown node order");
    if (ninst < 1) fail(PD_EINVAL, "need at least one instance");
    std::vector<Inst> insts(static_cast<size_t>(ninst));
    int64_t total = 0;
    for (int32_t b = 0; b < ninst; ++b) {
        validate_coords(n[b], coords[b], horizon[b]);
        Inst& I = insts[b];
        I.n = n[b];
        I.horizon = horizon[b];
        I.x.assign(coords[b], coords[b] + 3 * n[b]);
        if (user_row_ptr) {  // the caller's family (one instance), validated already
            I.row_ptr.assign(user_row_ptr, user_row_ptr + n[b] + 1);
            I.col.assign(user_col, user_col + user_row_ptr[n[b]]);
        } else {
            family_search(I.n, I.x.data(), I.horizon, I.row_ptr, I.col);
        }
        I.nnz = I.row_ptr[I.n];
        I.bc_kind.assign(static_cast<size_t>(3 * I.n), 0);
        I.bc_sched.assign(static_cast<size_t>(3 * I.n), 0);
        I.bc_val.assign(static_cast<size_t>(3 * I.n), 0.0);
        total += I.nnz;
    }
    (void)total;
    set_device(ctx);
    ctx->built = ctx->laid = ctx->recut = false;
    ctx->kept.reset();
    ctx->drop_graphs();
    ctx->tape_valid = false;
    ctx->inst = std::move(insts);
    ctx->order = order == PD_ORDER_AUTO ? PD_ORDER_NATURAL : order;
    ctx->order_auto = order == PD_ORDER_AUTO;
    ctx->has_nofail = false;
    ctx->has_laws = false;
    ctx->has_osb = false;
    ctx->adjoint = false;
    ctx->step = 0;
    ctx->a_valid = false;
    ctx->vv_ahead = false;
    const int W = ctx->mapping == PD_MAP_STAGED ? kWave : kWave / ctx->lanes;
    int64_t nn = 0;
    for (const Inst& I : ctx->inst) nn += (I.n + W - 1) / W * W;
    check_nodes(nn);
    ctx->built = true;
    upload_stiffness(ctx);  // (the flags of what a problem holds)
    upload_volumes(ctx);
    upload_node_weights(ctx);
    upload_body(ctx);
    upload_laws(ctx);
    upload_osb(ctx);
}

}  // namespace host
}  // namespace pdmi

