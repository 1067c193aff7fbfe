// mesh_store.cpp -- device mesh store: validation of a host mesh
// description, the processing order (tiles), the signed node->edge table in
// that order, and the one-time copy to the device.
//
// Section 4.3 (Block/Irregular connectivity: the node->edge table is an
// irregular table, edge2node a block table) and Section 5 (mesh data is
// made available on the device once, then stays resident).
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <exception>
#include <memory>
#include <numeric>
#include <string>
#include <thread>
#include <utility>
#include <vector>

#include "internal.h"

namespace atlasx {

MeshStore::~MeshStore() {
  for (void *p : allocations) (void)hipFree(p);
  if (ws) (void)hipFree(ws);
}

namespace {

atlas_status validate(const atlas_mesh_desc *d) {
  if (!d) return fail(ATLAS_EINVAL, "mesh description is NULL");
  const int64_t V = d->nnodes, E = d->nedges;
  if (V < 1 || V >= (int64_t)1 << 31)
    return fail(ATLAS_EINVAL, "nnodes must be in [1, 2^31)");
  if (E < 1 || 2 * E >= (int64_t)1 << 31)
    return fail(ATLAS_EINVAL, "nedges must be in [1, 2^30)");
  if (!d->lon || !d->lat || !d->cos_lat || !d->edge2node || !d->node2edge_ptr ||
      !d->node2edge || !d->node2edge_sign || !d->dual_volumes || !d->dual_normals)
    return fail(ATLAS_EINVAL, "a required mesh array is NULL");
  if (d->npole_edges < 0 || (d->npole_edges > 0 && (!d->pole_edges || !d->pole_normals)))
    return fail(ATLAS_EINVAL, "pole edge arrays missing");
  if (!(d->radius > 0.0) || !std::isfinite(d->radius))
    return fail(ATLAS_EINVAL, "radius must be positive and finite");
  for (int64_t e = 0; e < E; ++e) {
    const int32_t a = d->edge2node[2 * e], b = d->edge2node[2 * e + 1];
    if (a < 0 || b >= V || !(a < b))
      return fail(ATLAS_EINVAL, "edge2node[" + std::to_string(e) + "] must satisfy 0 <= a < b < nnodes");
    if (!std::isfinite(d->dual_normals[2 * e]) || !std::isfinite(d->dual_normals[2 * e + 1]))
      return fail(ATLAS_EINVAL, "non-finite dual normal at edge " + std::to_string(e));
  }
  if (d->node2edge_ptr[0] != 0 || d->node2edge_ptr[V] != 2 * E)
    return fail(ATLAS_EINVAL, "node2edge_ptr must run from 0 to 2*nedges");
  std::vector<uint8_t> seen(E, 0);
  for (int64_t i = 0; i < V; ++i) {
    const int64_t r0 = d->node2edge_ptr[i], r1 = d->node2edge_ptr[i + 1];
    if (r1 < r0) return fail(ATLAS_EINVAL, "node2edge_ptr is not monotone");
    for (int64_t r = r0; r < r1; ++r) {
      const int32_t e = d->node2edge[r];
      if (e < 0 || e >= E) return fail(ATLAS_EINVAL, "node2edge entry out of range");
      if (r > r0 && !(d->node2edge[r - 1] < e))
        return fail(ATLAS_EINVAL, "node2edge rows must list edges in ascending id");
      const int8_t s = d->node2edge_sign[r];
      const int32_t a = d->edge2node[2 * e], b = d->edge2node[2 * e + 1];
      if (!((s == 1 && a == i) || (s == -1 && b == i)))
        return fail(ATLAS_EINVAL, "node2edge_sign / endpoint mismatch at node " + std::to_string(i));
      seen[e] |= (s == 1) ? 1 : 2;
    }
    if (!(d->dual_volumes[i] > 0.0) || !std::isfinite(d->dual_volumes[i]))
      return fail(ATLAS_EINVAL, "dual volume must be positive at node " + std::to_string(i));
    if (!(d->cos_lat[i] > 0.0) || d->cos_lat[i] > 1.0 || !std::isfinite(d->lat[i]) ||
        !std::isfinite(d->lon[i]))
      return fail(ATLAS_EINVAL, "bad coordinates at node " + std::to_string(i));
  }
  for (int64_t e = 0; e < E; ++e)
    if (seen[e] != 3) return fail(ATLAS_EINVAL, "edge " + std::to_string(e) + " missing from node2edge");
  std::vector<uint8_t> polar(V, 0);
  for (int64_t k = 0; k < d->npole_edges; ++k) {
    const int32_t a = d->pole_edges[2 * k], b = d->pole_edges[2 * k + 1];
    if (a < 0 || b < 0 || a >= V || b >= V || a == b)
      return fail(ATLAS_EINVAL, "pole edge endpoints out of range");
    if (polar[a]++ || polar[b]++)
      return fail(ATLAS_EINVAL, "a node belongs to more than one pole edge");
    if (!std::isfinite(d->pole_normals[k])) return fail(ATLAS_EINVAL, "non-finite pole normal");
  }
  return ATLAS_OK;
}

// Parallels: explicit ring_off, or runs of equal latitude in node order.
std::vector<int64_t> rings_of(const atlas_mesh_desc *d) {
  std::vector<int64_t> off;
  if (d->nrings > 0 && d->ring_off) {
    off.assign(d->ring_off, d->ring_off + d->nrings + 1);
    bool ok = off.front() == 0 && off.back() == d->nnodes;
    for (size_t j = 0; ok && j + 1 < off.size(); ++j) ok = off[j] < off[j + 1];
    if (ok) return off;
    off.clear();
  }
  off.push_back(0);
  for (int64_t i = 1; i < d->nnodes; ++i)
    if (d->lat[i] != d->lat[i - 1]) off.push_back(i);
  off.push_back(d->nnodes);
  return off;
}

}  // namespace

bool zipper_conforming(const atlas_mesh_desc *d, const std::vector<int64_t> &off) {
  const int64_t nr = (int64_t)off.size() - 1;
  if (nr < 2) return false;
  const double twopi = 6.283185307179586476925;
  for (int64_t j = 0; j < nr; ++j) {
    const int64_t o = off[j], n = off[j + 1] - o;
    if (n < 3 || d->lon[o] != 0.0) return false;
    if (j > 0 && !(d->lat[o] < d->lat[off[j - 1]])) return false;
    for (int64_t i = 0; i < n; ++i) {
      if (d->lat[o + i] != d->lat[o]) return false;
      if (!(d->lon[o + i] < twopi) || (i > 0 && !(d->lon[o + i] > d->lon[o + i - 1])))
        return false;
    }
  }
  // is {p, q} an edge?  (scan the smaller node's CSR row)
  auto has_edge = [&](int64_t p, int64_t q) {
    const int64_t a = std::min(p, q), b = std::max(p, q);
    for (int64_t r = d->node2edge_ptr[a]; r < d->node2edge_ptr[a + 1]; ++r) {
      const int32_t e = d->node2edge[r];
      if (d->edge2node[2 * e] == a && d->edge2node[2 * e + 1] == b) return true;
    }
    return false;
  };
  int64_t count = 0;
  for (int64_t j = 0; j < nr; ++j) {  // edges along each parallel
    const int64_t o = off[j], n = off[j + 1] - o;
    for (int64_t i = 0; i < n; ++i)
      if (!has_edge(o + i, o + (i + 1) % n)) return false;
    count += n;
  }
  for (int64_t j = 0; j + 1 < nr; ++j) {  // edges across each strip, walked
    const int64_t ou = off[j], nu = off[j + 1] - ou;
    const int64_t ol = off[j + 1], nl = off[j + 2] - ol;
    int64_t a = 0, b = 0;
    while (a + b < nu + nl) {
      if (!has_edge(ou + a % nu, ol + b % nl)) return false;
      const bool up = a < nu && (b == nl || (a + 1) * nl < (b + 1) * nu ||
                                 ((a + 1) * nl == (b + 1) * nu && nu > nl));
      if (up) ++a; else ++b;
    }
    count += nu + nl;
  }
  return count == d->nedges;
}

// Processing order: bands of `band` parallels; each band is cut into
// longitude sectors holding about `width` nodes of its widest parallel;
// a tile is one sector of one band, listed parallel by parallel.  Meshes
// without a parallel structure fall back to blocks of consecutive nodes.
static void processing_order(const atlas_mesh_desc *d, int band, int width,
                             std::vector<int32_t> &perm, std::vector<int32_t> &tile_ptr,
                             int32_t &nrings) {
  const int64_t V = d->nnodes;
  std::vector<int64_t> off = rings_of(d);
  const int64_t nr = (int64_t)off.size() - 1;
  nrings = (int32_t)nr;
  perm.clear();
  perm.reserve(V);
  tile_ptr.assign(1, 0);
  if (nr > V / 4) {
    for (int64_t i = 0; i < V; ++i) {
      perm.push_back((int32_t)i);
      if ((i + 1) % (band * width) == 0 || i + 1 == V) tile_ptr.push_back((int32_t)(i + 1));
    }
    return;
  }
  const double twopi = 6.283185307179586476925;
  for (int64_t j0 = 0; j0 < nr; j0 += band) {
    const int64_t j1 = std::min(nr, j0 + band);
    int64_t widest = 0;
    for (int64_t j = j0; j < j1; ++j) widest = std::max(widest, off[j + 1] - off[j]);
    const int64_t nsec = std::max<int64_t>(1, (widest + width / 2) / width);
    std::vector<std::vector<int32_t>> bucket(nsec);
    for (int64_t j = j0; j < j1; ++j) {
      for (int64_t i = off[j]; i < off[j + 1]; ++i) {
        double x = std::fmod(d->lon[i], twopi);
        if (x < 0) x += twopi;
        int64_t sec = (int64_t)(x / twopi * (double)nsec);
        if (sec >= nsec) sec = nsec - 1;
        bucket[sec].push_back((int32_t)i);
      }
    }
    for (int64_t s = 0; s < nsec; ++s) {
      perm.insert(perm.end(), bucket[s].begin(), bucket[s].end());
      if ((int64_t)perm.size() > tile_ptr.back()) tile_ptr.push_back((int32_t)perm.size());
    }
  }
}

// Work over `n` tiles on the host's threads: how many to use (eight tiles each
// at least, some eight thousand nodes), and fn(w) for w = 0 .. count - 1 on
// them.
static int host_threads(int64_t n) {
  const int64_t hw = std::max(1u, std::thread::hardware_concurrency());
  return (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(hw, 16), n / 8));
}
template <class F>
static void on_threads(int count, const F &fn) {
  std::vector<std::exception_ptr> err(count);
  auto run = [&](int w) {
    try {
      fn(w);
    } catch (...) {  // rethrown below, on the calling thread
      err[w] = std::current_exception();
    }
  };
  std::vector<std::thread> th;
  th.reserve(count);
  int started = 1;
  try {
    for (; started < count; ++started) th.emplace_back(run, started);
  } catch (...) {  // no more threads to be had: the rest runs here
  }
  run(0);
  for (int w = started; w < count; ++w) run(w);
  for (auto &t : th) t.join();
  for (auto &e : err)
    if (e) std::rethrow_exception(e);
}

// Indices of nodes on a parallel, as bits: a plan adds every neighbour of a
// tile's nodes, each some seven times over, and asks for the run that holds
// them (lists sorted and made unique took most of an upload).
struct RunSet {
  std::vector<uint64_t> bits;
  std::vector<int32_t> words;  // the words with bits set
  void add(int32_t i) {
    const size_t w = (size_t)i >> 6;
    if (w >= bits.size()) bits.resize(w + 1, 0);
    if (!bits[w]) words.push_back((int32_t)w);
    bits[w] |= (uint64_t)1 << (i & 63);
  }
  // The shortest cyclic run of a parallel of nx nodes that holds the indices,
  // the complement of their widest gap; the set is empty afterwards.  False
  // if the run's slots would not fit 16 bits.
  bool run(int32_t nx, int32_t &lo, int32_t &len) {
    std::sort(words.begin(), words.end());
    int32_t count = 0, first = 0, last = 0, best = -1, after = 0;
    for (int32_t w : words) {
      for (uint64_t b = bits[w]; b; b &= b - 1) {
        const int32_t i = w * 64 + __builtin_ctzll(b);
        if (count++ == 0) {
          first = i;
        } else if (i - last > best) {
          best = i - last;
          after = i;
        }
        last = i;
      }
      bits[w] = 0;
    }
    words.clear();
    if (count == 0 || count == nx) {
      lo = 0;
      len = count;
    } else {
      if (first + nx - last > best) {
        best = first + nx - last;
        after = first;
      }
      lo = after;
      len = nx - best + 1;
    }
    return len < 65536;
  }
};

// Parallel-sweep plan.  For every tile: the parallels it owns plus one
// above and one below, each reduced to the shortest cyclic run of nodes that
// holds the tile's own nodes and all their neighbours; the slot of every
// position in its run and of every neighbour in its run.  A kernel keeps
// the runs of three consecutive parallels in LDS and reads every neighbour
// from there.  Returns false if a neighbour lies more than one parallel away
// (then the plan is not used).
struct SweepPlan {
  std::vector<int32_t> tile_seg, selfslot, lref;
  std::vector<int4> seg;
  std::vector<int2> seg_pos;
  int32_t segmax = 0;
};

static bool sweep_plan(const std::vector<int64_t> &off, const std::vector<int32_t> &perm,
                       const std::vector<int32_t> &tile_ptr, const std::vector<int32_t> &rowp,
                       const std::vector<int32_t> &nbr, SweepPlan &sp) {
  const int64_t V = (int64_t)perm.size();
  const int64_t nr = (int64_t)off.size() - 1;
  std::vector<int32_t> ring_of(V);
  for (int64_t j = 0; j < nr; ++j)
    for (int64_t i = off[j]; i < off[j + 1]; ++i) ring_of[i] = (int32_t)j;
  const int64_t T = (int64_t)tile_ptr.size() - 1;
  sp.tile_seg.assign(1, 0);
  sp.selfslot.assign(V, 0);
  sp.lref.assign(nbr.size(), -1);
  std::vector<RunSet> need;
  for (int64_t t = 0; t < T; ++t) {
    const int32_t p0 = tile_ptr[t], p1 = tile_ptr[t + 1];
    int32_t jmin = INT32_MAX, jmax = -1;
    for (int32_t p = p0; p < p1; ++p) {
      const int32_t j = ring_of[perm[p]];
      if (p > p0 && j < ring_of[perm[p - 1]]) return false;  // parallels in order
      jmin = std::min(jmin, j);
      jmax = std::max(jmax, j);
    }
    const int32_t rlo = std::max<int32_t>(0, jmin - 1);
    const int32_t rhi = std::min<int32_t>((int32_t)nr - 1, jmax + 1);
    if ((int64_t)need.size() < rhi - rlo + 1) need.resize(rhi - rlo + 1);
    std::vector<int2> pos(rhi - rlo + 1, make_int2(0, 0));
    for (int32_t p = p0; p < p1; ++p) {
      const int32_t i = perm[p], j = ring_of[i];
      need[j - rlo].add((int32_t)(i - off[j]));
      if (pos[j - rlo].y == 0) pos[j - rlo] = make_int2(p, p + 1);
      else pos[j - rlo].y = p + 1;
      for (int32_t r = rowp[p]; r < rowp[p + 1]; ++r) {
        const int32_t n = (int32_t)((uint32_t)nbr[r] & ~kPoleBit), jn = ring_of[n];
        if (jn < j - 1 || jn > j + 1) return false;
        need[jn - rlo].add((int32_t)(n - off[jn]));
      }
    }
    std::vector<int32_t> lo(rhi - rlo + 1), len(rhi - rlo + 1);
    for (int32_t q = 0; q <= rhi - rlo; ++q) {
      const int32_t nx = (int32_t)(off[rlo + q + 1] - off[rlo + q]);
      if (!need[q].run(nx, lo[q], len[q])) return false;
      sp.segmax = std::max(sp.segmax, len[q]);
      sp.seg.push_back(make_int4((int32_t)off[rlo + q], nx, lo[q], len[q]));
      sp.seg_pos.push_back(pos[q]);
    }
    sp.tile_seg.push_back((int32_t)sp.seg.size());
    auto slot = [&](int32_t node, int32_t q) {
      const int32_t nx = (int32_t)(off[rlo + q + 1] - off[rlo + q]);
      int32_t s = (int32_t)(node - off[rlo + q]) - lo[q];
      if (s < 0) s += nx;
      return s;
    };
    for (int32_t p = p0; p < p1; ++p) {
      const int32_t i = perm[p], q = ring_of[i] - rlo;
      sp.selfslot[p] = slot(i, q);
      for (int32_t r = rowp[p]; r < rowp[p + 1]; ++r) {
        const bool pole = ((uint32_t)nbr[r] & kPoleBit) != 0;
        const int32_t n = (int32_t)((uint32_t)nbr[r] & ~kPoleBit);
        const int32_t qn = ring_of[n] - rlo;
        const int32_t s = slot(n, qn);
        if (s >= len[qn]) return false;
        sp.lref[r] = (pole ? kLrefPole : 0) | ((qn - q + 1) << 16) | s;
      }
    }
  }
  return true;
}

// The sweep's tiles cut into `parts` longitude parts (part k owns the k-th
// share of the tile's positions on every parallel) and their bands into
// `bands`.  Like sweep_plan per piece, with the references as rows of the
// ring the wave-specialised sweep keeps its runs in.  False where a reference
// would not fit its 16 bits or a row has more than six incidences.
struct CutPlan {
  std::vector<int32_t> tile_seg;
  std::vector<int4> seg, refs;
  std::vector<int2> seg_pos;
  int32_t segmax = 0, pmax = 0, rings = 0;
};

static bool cut_plan(const std::vector<int64_t> &off, const std::vector<int32_t> &ring_of,
                     const std::vector<int32_t> &perm, const std::vector<int32_t> &tile_ptr,
                     const std::vector<int32_t> &rowp, const std::vector<int32_t> &nbr, int parts,
                     int bands, CutPlan &cp) {
  const int64_t T = (int64_t)tile_ptr.size() - 1;
  const int32_t nr = (int32_t)off.size() - 1;
  auto nb = [&](int32_t r) { return (int32_t)((uint32_t)nbr[r] & ~kPoleBit); };
  // every thread takes a range of tiles and lists their runs
  struct Part {
    std::vector<int32_t> nseg;  // runs of each tile part
    std::vector<int4> seg;
    std::vector<int2> seg_pos;
    int32_t segmax = 0, pmax = 0, rings = 0;
    bool ok = true;
  };
  const int pieces = parts * bands;
  const int nthr = host_threads(T);
  std::vector<Part> done(nthr);
  auto runs = [&](int w) {
    Part &o = done[w];
    std::vector<int2> own, pos;
    std::vector<RunSet> need;
    for (int64_t t = T * w / nthr; t < T * (w + 1) / nthr && o.ok; ++t) {
      // the tile's positions on each of its parallels
      const int32_t j0 = ring_of[perm[tile_ptr[t]]];
      own.clear();
      for (int32_t p = tile_ptr[t]; p < tile_ptr[t + 1]; ++p) {
        const int32_t q = ring_of[perm[p]] - j0;
        while ((int32_t)own.size() <= q) own.push_back(make_int2(p, p));
        own[q].y = p + 1;
      }
      for (int u = 0; u < pieces; ++u) {
        const int k = u % parts, b = u / parts;
        const int64_t nq = (int64_t)own.size();
        const int32_t qa = (int32_t)(nq * b / bands), qb = (int32_t)(nq * (b + 1) / bands);
        o.rings = std::max(o.rings, qb - qa);
        const int32_t rlo = std::max(0, j0 + qa - 1), rhi = std::min(nr - 1, j0 + qb);
        if ((int64_t)need.size() < rhi - rlo + 1) need.resize(rhi - rlo + 1);
        pos.assign(rhi - rlo + 1, make_int2(0, 0));
        for (int32_t q = qa; q < qb; ++q) {
          const int32_t n = own[q].y - own[q].x;
          const int2 pr = make_int2(own[q].x + (int32_t)((int64_t)n * k / parts),
                                    own[q].x + (int32_t)((int64_t)n * (k + 1) / parts));
          pos[j0 + q - rlo] = pr;
          o.pmax = std::max(o.pmax, pr.y - pr.x);
          for (int32_t p = pr.x; p < pr.y; ++p) {
            need[j0 + q - rlo].add((int32_t)(perm[p] - off[j0 + q]));
            if (rowp[p + 1] - rowp[p] > 6) o.ok = false;
            for (int32_t r = rowp[p]; r < rowp[p + 1]; ++r)
              need[ring_of[nb(r)] - rlo].add((int32_t)(nb(r) - off[ring_of[nb(r)]]));
          }
        }
        o.nseg.push_back(rhi - rlo + 1);
        for (int32_t q = 0; q <= rhi - rlo; ++q) {
          const int32_t nx = (int32_t)(off[rlo + q + 1] - off[rlo + q]);
          int32_t lo = 0, len = 0;
          if (!need[q].run(nx, lo, len)) o.ok = false;
          o.segmax = std::max(o.segmax, len);
          o.seg.push_back(make_int4((int32_t)off[rlo + q], nx, lo, len));
          o.seg_pos.push_back(pos[q]);
        }
      }
    }
  };
  on_threads(nthr, runs);
  cp.tile_seg.assign(1, 0);
  std::vector<size_t> base(nthr, 0);
  for (int w = 0; w < nthr; ++w) {
    const Part &o = done[w];
    if (!o.ok) return false;
    base[w] = cp.seg.size();
    for (int32_t n : o.nseg) cp.tile_seg.push_back(cp.tile_seg.back() + n);
    cp.seg.insert(cp.seg.end(), o.seg.begin(), o.seg.end());
    cp.seg_pos.insert(cp.seg_pos.end(), o.seg_pos.begin(), o.seg_pos.end());
    cp.segmax = std::max(cp.segmax, o.segmax);
    cp.pmax = std::max(cp.pmax, o.pmax);
    cp.rings = std::max(cp.rings, o.rings);
  }
  if ((int64_t)kSweepwSlots * cp.segmax >= 65536) return false;
  cp.refs.resize(perm.size());
  on_threads(nthr, [&](int w) {
    for (int64_t u = T * w / nthr * pieces; u < T * (w + 1) / nthr * pieces; ++u) {
      const int32_t s0 = cp.tile_seg[u], s1 = cp.tile_seg[u + 1];
      for (int32_t s = s0; s < s1; ++s) {
        // ring row of node i, on the parallel of run s + dq
        auto row = [&](int32_t i, int32_t dq) {
          const int4 g = cp.seg[s + dq];
          int32_t t = i - g.x - g.z;
          if (t < 0) t += g.y;
          return (s + dq - s0) % kSweepwSlots * cp.segmax + t;
        };
        for (int32_t p = cp.seg_pos[s].x; p < cp.seg_pos[s].y; ++p) {
          const int32_t n = rowp[p + 1] - rowp[p], j = ring_of[perm[p]];
          const int32_t self = row(perm[p], 0);
          int32_t r[6], flags = n << 16;
          for (int32_t k = 0; k < 6; ++k) {
            r[k] = self;
            if (k >= n) continue;
            r[k] = row(nb(rowp[p] + k), ring_of[nb(rowp[p] + k)] - j);
            if ((uint32_t)nbr[rowp[p] + k] & kPoleBit) flags |= kSgeoPole << k;
          }
          if (n == 6 && !(flags & (63 * kSgeoPole))) flags |= kSgeoFull;
          cp.refs[p] = make_int4(self | flags, r[0] | r[1] << 16, r[2] | r[3] << 16,
                                 r[4] | r[5] << 16);
        }
      }
    }
  });
  return true;
}

// Two-ring plan of the fused Laplacian.  For every tile: its own
// parallels [ja, jb]; the gradient is needed at the tile's nodes and their
// neighbours (parallels ja-1 .. jb+1), and those gradients need the field at
// their own neighbours (parallels ja-2 .. jb+2).  Per parallel of that
// window: the f-run (shortest cyclic run holding every node whose field is
// read), the g-run (the same for the nodes whose gradient is formed; every
// node of the g-run gets one, so all of them are covered by the f-runs), and
// the tile's own positions.  Per g-run node: its incidence row start, count,
// its slot in its f-run and its neighbours' f-run slots; per own position:
// its slot in its g-run and its neighbours' g-run slots.  References are
// ((dq + 1) << 16) | slot (dq = neighbour parallel - own parallel) plus
// kLrefPole for a pole edge.  Returns false if a neighbour lies more than
// one parallel away.
struct LaplPlan {
  std::vector<int32_t> tile_seg;  // [T+1] window range of a tile in fseg/gseg
  std::vector<int4> fseg;         // {ring offset, ring size, f-run first, f-run length}
  std::vector<int4> gseg;         // {g-run first, g-run length, first g record, 0}
  std::vector<int2> seg_pos;      // own positions on the parallel [lo, hi)
  std::vector<int4> gnode;        // per g record {row start, row length, f self slot, position}
  std::vector<int32_t> glref;     // per g record: kGRefs references into the f-runs
  std::vector<int32_t> lref;      // per incidence (own positions): into the g-runs
  std::vector<int32_t> lself;     // per position: slot in its g-run
  int32_t fmax = 0, gmax = 0, pmax = 0;
};

static bool lapl_plan(const std::vector<int64_t> &off, const std::vector<int32_t> &ring_of,
                      const std::vector<int32_t> &perm, const std::vector<int32_t> &inv,
                      const std::vector<int32_t> &tile_ptr, const std::vector<int32_t> &rowp,
                      const std::vector<int32_t> &nbr, LaplPlan &lp) {
  const int64_t V = (int64_t)perm.size();
  const int32_t nr = (int32_t)off.size() - 1;
  const int64_t T = (int64_t)tile_ptr.size() - 1;
  lp.tile_seg.assign(1, 0);
  lp.lref.assign(nbr.size(), 1 << 16);
  lp.lself.assign(V, 0);
  auto nb = [&](int32_t r) { return (int32_t)((uint32_t)nbr[r] & ~kPoleBit); };
  std::vector<RunSet> gneed, fneed;
  for (int64_t t = 0; t < T; ++t) {
    const int32_t p0 = tile_ptr[t], p1 = tile_ptr[t + 1];
    int32_t ja = INT32_MAX, jb = -1;
    for (int32_t p = p0; p < p1; ++p) {
      const int32_t j = ring_of[perm[p]];
      if (p > p0 && j < ring_of[perm[p - 1]]) return false;  // parallels in order
      ja = std::min(ja, j);
      jb = std::max(jb, j);
    }
    const int32_t rlo = std::max(0, ja - 2), rhi = std::min(nr - 1, jb + 2);
    const int32_t W = rhi - rlo + 1;
    if ((int64_t)gneed.size() < W) {
      gneed.resize(W);
      fneed.resize(W);
    }
    std::vector<int2> pos(W, make_int2(0, 0));
    auto local = [&](int32_t node) { return (int32_t)(node - off[ring_of[node]]); };
    for (int32_t p = p0; p < p1; ++p) {
      const int32_t i = perm[p], j = ring_of[i];
      gneed[j - rlo].add(local(i));
      if (pos[j - rlo].y == 0) pos[j - rlo] = make_int2(p, p + 1);
      else pos[j - rlo].y = p + 1;
      for (int32_t r = rowp[p]; r < rowp[p + 1]; ++r) {
        const int32_t n = nb(r), jn = ring_of[n];
        if (jn < j - 1 || jn > j + 1) return false;
        gneed[jn - rlo].add(local(n));
      }
    }
    std::vector<int32_t> glo(W), glen(W), flo(W), flen(W);
    for (int32_t q = 0; q < W; ++q) {
      const int32_t nx = (int32_t)(off[rlo + q + 1] - off[rlo + q]);
      if (!gneed[q].run(nx, glo[q], glen[q])) return false;
      // every node of the g-run gets a gradient: its field and its
      // neighbours' fields are read
      for (int32_t s = 0; s < glen[q]; ++s) {
        const int32_t i = (int32_t)off[rlo + q] + (glo[q] + s) % nx;
        const int32_t p = inv[i], j = rlo + q;
        fneed[q].add(local(i));
        for (int32_t r = rowp[p]; r < rowp[p + 1]; ++r) {
          const int32_t n = nb(r), jn = ring_of[n];
          if (jn < j - 1 || jn > j + 1 || jn < rlo || jn > rhi) return false;
          fneed[jn - rlo].add(local(n));
        }
      }
    }
    for (int32_t q = 0; q < W; ++q) {
      const int32_t nx = (int32_t)(off[rlo + q + 1] - off[rlo + q]);
      if (!fneed[q].run(nx, flo[q], flen[q])) return false;
    }
    auto fslot = [&](int32_t node) {
      const int32_t q = ring_of[node] - rlo;
      const int32_t nx = (int32_t)(off[rlo + q + 1] - off[rlo + q]);
      int32_t s = local(node) - flo[q];
      if (s < 0) s += nx;
      return s;
    };
    auto gslot = [&](int32_t node) {
      const int32_t q = ring_of[node] - rlo;
      const int32_t nx = (int32_t)(off[rlo + q + 1] - off[rlo + q]);
      int32_t s = local(node) - glo[q];
      if (s < 0) s += nx;
      return s;
    };
    for (int32_t q = 0; q < W; ++q) {
      const int32_t nx = (int32_t)(off[rlo + q + 1] - off[rlo + q]);
      lp.fmax = std::max(lp.fmax, flen[q]);
      lp.gmax = std::max(lp.gmax, glen[q]);
      lp.pmax = std::max(lp.pmax, pos[q].y - pos[q].x);
      lp.fseg.push_back(make_int4((int32_t)off[rlo + q], nx, flo[q], flen[q]));
      lp.gseg.push_back(make_int4(glo[q], glen[q], (int32_t)lp.gnode.size(), 0));
      lp.seg_pos.push_back(pos[q]);
      const int32_t j = rlo + q;
      for (int32_t s = 0; s < glen[q]; ++s) {
        const int32_t i = (int32_t)off[j] + (glo[q] + s) % nx;
        const int32_t p = inv[i], n0 = rowp[p], n1 = rowp[p + 1];
        if (n1 - n0 > kGRefs) return false;
        const int32_t self = fslot(i);
        if (self >= flen[q]) return false;
        lp.gnode.push_back(make_int4(n0, n1 - n0, self, p));
        for (int32_t k = 0; k < kGRefs; ++k) {
          int32_t ref = 1 << 16;  // padding: the own parallel, slot 0
          if (k < n1 - n0) {
            const int32_t r = n0 + k, n = nb(r), qn = ring_of[n] - rlo;
            const int32_t sl = fslot(n);
            if (sl >= flen[qn]) return false;
            ref = ((((uint32_t)nbr[r] & kPoleBit) != 0) ? kLrefPole : 0) |
                  ((ring_of[n] - j + 1) << 16) | sl;
          }
          lp.glref.push_back(ref);
        }
      }
    }
    for (int32_t p = p0; p < p1; ++p) {
      const int32_t i = perm[p], j = ring_of[i];
      lp.lself[p] = gslot(i);
      if (lp.lself[p] >= glen[j - rlo]) return false;
      for (int32_t r = rowp[p]; r < rowp[p + 1]; ++r) {
        const int32_t n = nb(r), qn = ring_of[n] - rlo;
        const int32_t sl = gslot(n);
        if (sl >= glen[qn]) return false;
        lp.lref[r] = ((((uint32_t)nbr[r] & kPoleBit) != 0) ? kLrefPole : 0) |
                     ((ring_of[n] - j + 1) << 16) | sl;
      }
    }
    lp.tile_seg.push_back((int32_t)lp.fseg.size());
  }
  return true;
}

// The fused Laplacian's pieces (tiles cut as in cut_plan) on the two-ring
// window of lapl_plan, with references as ring rows.  False as for cut_plan.
struct LaplCutPlan {
  std::vector<int32_t> tile_seg;
  std::vector<int4> fseg, gseg, grefs, orefs;
  std::vector<int2> seg_pos;
  int32_t fmax = 1, gmax = 1, pmax = 1, rings = 0;
};

static bool lapl_cut_plan(const std::vector<int64_t> &off, const std::vector<int32_t> &ring_of,
                          const std::vector<int32_t> &perm, const std::vector<int32_t> &inv,
                          const std::vector<int32_t> &tile_ptr, const std::vector<int32_t> &rowp,
                          const std::vector<int32_t> &nbr, int parts, int bands, LaplCutPlan &lp) {
  const int64_t T = (int64_t)tile_ptr.size() - 1;
  const int32_t nr = (int32_t)off.size() - 1;
  auto nb = [&](int32_t r) { return (int32_t)((uint32_t)nbr[r] & ~kPoleBit); };
  struct Part {
    std::vector<int32_t> nseg;
    std::vector<int4> fseg, gseg;  // (gseg.z: g nodes before this one in the part)
    std::vector<int2> seg_pos;
    int32_t fmax = 1, gmax = 1, pmax = 1, rings = 0, ng = 0;
    bool ok = true;
  };
  const int pieces = parts * bands;
  const int nthr = host_threads(T);
  std::vector<Part> done(nthr);
  on_threads(nthr, [&](int w) {
    Part &o = done[w];
    std::vector<int2> own;
    std::vector<RunSet> gneed, fneed;
    for (int64_t t = T * w / nthr; t < T * (w + 1) / nthr && o.ok; ++t) {
      const int32_t j0 = ring_of[perm[tile_ptr[t]]];
      own.clear();
      for (int32_t p = tile_ptr[t]; p < tile_ptr[t + 1]; ++p) {
        const int32_t q = ring_of[perm[p]] - j0;
        while ((int32_t)own.size() <= q) own.push_back(make_int2(p, p));
        own[q].y = p + 1;
      }
      for (int u = 0; u < pieces; ++u) {
        const int k = u % parts, b = u / parts;
        const int64_t nq = (int64_t)own.size();
        const int32_t qa = (int32_t)(nq * b / bands), qb = (int32_t)(nq * (b + 1) / bands);
        o.rings = std::max(o.rings, qb - qa);
        const int32_t rlo = std::max(0, j0 + qa - 2), rhi = std::min(nr - 1, j0 + qb + 1);
        const int32_t W = rhi - rlo + 1;
        if ((int64_t)gneed.size() < W) {
          gneed.resize(W);
          fneed.resize(W);
        }
        const size_t s0 = o.seg_pos.size();
        for (int32_t q = 0; q < W; ++q) o.seg_pos.push_back(make_int2(0, 0));
        for (int32_t q = qa; q < qb; ++q) {
          const int32_t n = own[q].y - own[q].x, j = j0 + q;
          const int2 pr = make_int2(own[q].x + (int32_t)((int64_t)n * k / parts),
                                    own[q].x + (int32_t)((int64_t)n * (k + 1) / parts));
          o.seg_pos[s0 + j - rlo] = pr;
          o.pmax = std::max(o.pmax, pr.y - pr.x);
          for (int32_t p = pr.x; p < pr.y; ++p) {
            gneed[j - rlo].add((int32_t)(perm[p] - off[j]));
            for (int32_t r = rowp[p]; r < rowp[p + 1]; ++r)  // (no pole edge in a divergence)
              if (!((uint32_t)nbr[r] & kPoleBit))
                gneed[ring_of[nb(r)] - rlo].add((int32_t)(nb(r) - off[ring_of[nb(r)]]));
          }
        }
        o.nseg.push_back(W);
        for (int32_t q = 0; q < W; ++q) {
          const int32_t j = rlo + q, nx = (int32_t)(off[j + 1] - off[j]);
          int32_t lo = 0, len = 0;
          if (!gneed[q].run(nx, lo, len)) o.ok = false;
          o.gmax = std::max(o.gmax, len);
          o.gseg.push_back(make_int4(lo, len, o.ng, 0));
          o.ng += len;
          // every node of the g-run gets a gradient
          for (int32_t s = 0; s < len; ++s) {
            const int32_t i = (int32_t)off[j] + (lo + s) % nx, p = inv[i];
            fneed[q].add(i - (int32_t)off[j]);
            if (rowp[p + 1] - rowp[p] > 6) o.ok = false;
            for (int32_t r = rowp[p]; r < rowp[p + 1]; ++r) {
              const int32_t jn = ring_of[nb(r)];
              if (jn < rlo || jn > rhi) {
                o.ok = false;
                break;
              }
              fneed[jn - rlo].add((int32_t)(nb(r) - off[jn]));
            }
          }
        }
        for (int32_t q = 0; q < W; ++q) {
          const int32_t nx = (int32_t)(off[rlo + q + 1] - off[rlo + q]);
          int32_t lo = 0, len = 0;
          if (!fneed[q].run(nx, lo, len)) o.ok = false;
          o.fmax = std::max(o.fmax, len);
          o.fseg.push_back(make_int4((int32_t)off[rlo + q], nx, lo, len));
        }
      }
    }
  });
  lp.tile_seg.assign(1, 0);
  int64_t ng = 0;
  for (const Part &o : done) {
    if (!o.ok) return false;
    for (int32_t n : o.nseg) lp.tile_seg.push_back(lp.tile_seg.back() + n);
    lp.fseg.insert(lp.fseg.end(), o.fseg.begin(), o.fseg.end());
    for (int4 g : o.gseg) lp.gseg.push_back(make_int4(g.x, g.y, g.z + (int32_t)ng, 0));
    lp.seg_pos.insert(lp.seg_pos.end(), o.seg_pos.begin(), o.seg_pos.end());
    lp.fmax = std::max(lp.fmax, o.fmax);
    lp.gmax = std::max(lp.gmax, o.gmax);
    lp.pmax = std::max(lp.pmax, o.pmax);
    lp.rings = std::max(lp.rings, o.rings);
    ng += o.ng;
    if (ng >= INT32_MAX) return false;
  }
  if ((int64_t)kLswFieldSlots * lp.fmax >= 65536 || (int64_t)kLswGradSlots * lp.gmax >= 65536)
    return false;
  lp.grefs.resize((size_t)ng);
  lp.orefs.resize(perm.size());
  on_threads(nthr, [&](int w) {
    for (int64_t u = T * w / nthr * pieces; u < T * (w + 1) / nthr * pieces; ++u) {
      const int32_t s0 = lp.tile_seg[u], s1 = lp.tile_seg[u + 1];
      for (int32_t s = s0; s < s1; ++s) {
        // the references of position p on the parallel of run s: rows of
        // the ring of f-runs (grad) or g-runs
        auto refs = [&](int32_t p, bool grad) {
          auto row = [&](int32_t i, int32_t dq) {
            const int4 f = lp.fseg[s + dq];
            int32_t t = i - f.x - (grad ? f.z : lp.gseg[s + dq].x);
            if (t < 0) t += f.y;
            return grad ? (s + dq - s0) % kLswFieldSlots * lp.fmax + t
                        : (s + dq - s0) % kLswGradSlots * lp.gmax + t;
          };
          const int32_t n = rowp[p + 1] - rowp[p], j = ring_of[perm[p]];
          const int32_t self = row(perm[p], 0);
          int32_t r[6], flags = n << 16;
          for (int32_t k = 0; k < 6; ++k) {
            r[k] = self;
            if (k >= n) continue;
            const bool pole = ((uint32_t)nbr[rowp[p] + k] & kPoleBit) != 0;
            if (pole) flags |= kSgeoPole << k;
            // (a pole edge does not enter the divergence, and its far end
            // need not be in the g-run)
            if (grad || !pole) r[k] = row(nb(rowp[p] + k), ring_of[nb(rowp[p] + k)] - j);
          }
          if (n == 6 && !(flags & (63 * kSgeoPole))) flags |= kSgeoFull;
          return make_int4(self | flags, r[0] | r[1] << 16, r[2] | r[3] << 16, r[4] | r[5] << 16);
        };
        const int4 f = lp.fseg[s], g = lp.gseg[s];
        for (int32_t t = 0; t < g.y; ++t)
          lp.grefs[g.z + t] = refs(inv[f.x + (g.x + t) % f.y], true);
        for (int32_t p = lp.seg_pos[s].x; p < lp.seg_pos[s].y; ++p) lp.orefs[p] = refs(p, false);
      }
    }
  });
  return true;
}

// Arrays on their way to the device: one allocation for all of them, and one
// copy for all but large ones (an allocation and a copy for each array took
// most of a small mesh's upload: O16 2.7 ms, 0.9 so).
class Upload {
 public:
  template <class T>
  void add(const std::vector<T> &h, const T **dptr) {
    items_.push_back({h.data(), h.size() * sizeof(T), total_, dptr});
    total_ += (h.size() * sizeof(T) + 255) / 256 * 256;
  }
  // *block: the allocation (the caller's to free); nothing is left on failure
  atlas_status commit(void **block) {
    void *p = nullptr;
    if (hipMalloc(&p, std::max<size_t>(256, total_)) != hipSuccess) {
      (void)hipGetLastError();
      return fail(ATLAS_ENOMEM, "hipMalloc of mesh store failed");
    }
    auto give_back = [](void *q) { (void)hipFree(q); };
    std::unique_ptr<void, decltype(give_back)> held(p, give_back);
    const atlas_status st = copy(static_cast<char *>(p));  // (may run out of host memory)
    if (st == ATLAS_OK) *block = held.release();
    return st;
  }
  size_t bytes() const { return std::max<size_t>(256, total_); }

 private:
  atlas_status copy(char *base) {
    constexpr size_t kLarge = (size_t)1 << 20;
    for (size_t k = 0; k < items_.size();) {
      // a run of smaller arrays goes by way of one host buffer
      size_t e = k;
      while (e < items_.size() && items_[e].bytes <= kLarge) ++e;
      if (e > k) {
        const size_t first = items_[k].offset;
        std::vector<char> buf(items_[e - 1].offset + items_[e - 1].bytes - first);
        for (size_t i = k; i < e; ++i)
          if (items_[i].bytes)
            std::memcpy(buf.data() + (items_[i].offset - first), items_[i].src, items_[i].bytes);
        if (!buf.empty())
          ATLASX_HIP(hipMemcpy(base + first, buf.data(), buf.size(), hipMemcpyHostToDevice));
        k = e;
      } else {
        ATLASX_HIP(hipMemcpy(base + items_[k].offset, items_[k].src, items_[k].bytes,
                             hipMemcpyHostToDevice));
        ++k;
      }
    }
    for (const Item &it : items_) {
      const void *q = base + it.offset;
      std::memcpy(it.dptr, &q, sizeof(q));
    }
    return ATLAS_OK;
  }
  struct Item {
    const void *src;
    size_t bytes, offset;
    void *dptr;  // the typed pointer to set
  };
  std::vector<Item> items_;
  size_t total_ = 0;
};

atlas_status upload_mesh(const atlas_mesh_desc *d, int band, int width, MeshStore **out) {
  atlas_status st = validate(d);
  if (st != ATLAS_OK) return st;
  const int64_t V = d->nnodes, E = d->nedges, NP = d->npole_edges;

  std::vector<int32_t> perm, tile_ptr;
  int32_t nrings = 0;
  processing_order(d, band, width, perm, tile_ptr, nrings);
  if ((int64_t)perm.size() != V) return fail(ATLAS_EINVAL, "processing order lost nodes");

  std::vector<int32_t> pole_of(V, -1);
  for (int64_t k = 0; k < NP; ++k) {
    pole_of[d->pole_edges[2 * k]] = (int32_t)k;
    pole_of[d->pole_edges[2 * k + 1]] = (int32_t)k;
  }
  // incidences in processing order: mesh edges in ascending id, pole last
  std::vector<int32_t> rowp(V + 1, 0), nbr, inc_edge;
  std::vector<double2> S;
  std::vector<double> vol_p(V), cos_p(V);
  nbr.reserve(2 * E + 2 * NP);
  inc_edge.reserve(2 * E + 2 * NP);
  S.reserve(2 * E + 2 * NP);
  int32_t maxdeg = 0, mindeg = INT32_MAX;
  for (int64_t p = 0; p < V; ++p) {
    const int32_t i = perm[p];
    mindeg = std::min<int32_t>(mindeg, (int32_t)(d->node2edge_ptr[i + 1] - d->node2edge_ptr[i]));
    for (int64_t r = d->node2edge_ptr[i]; r < d->node2edge_ptr[i + 1]; ++r) {
      const int32_t e = d->node2edge[r];
      const int8_t s = d->node2edge_sign[r];
      const int32_t other = s > 0 ? d->edge2node[2 * e + 1] : d->edge2node[2 * e];
      nbr.push_back(other);
      inc_edge.push_back(s > 0 ? e : (int32_t)(e | (int32_t)kPoleBit));
      S.push_back(make_double2(s * d->dual_normals[2 * e], s * d->dual_normals[2 * e + 1]));
    }
    if (pole_of[i] >= 0) {
      const int32_t k = pole_of[i];
      const int32_t a = d->pole_edges[2 * k], b = d->pole_edges[2 * k + 1];
      nbr.push_back((int32_t)((uint32_t)(a == i ? b : a) | kPoleBit));
      inc_edge.push_back((int32_t)(E + k));
      S.push_back(make_double2(0.0, d->pole_normals[k]));
    }
    rowp[p + 1] = (int32_t)nbr.size();
    maxdeg = std::max(maxdeg, rowp[p + 1] - rowp[p]);
    vol_p[p] = d->dual_volumes[i];
    cos_p[p] = d->cos_lat[i];
  }
  if (maxdeg > 64) return fail(ATLAS_EINVAL, "node degree above 64");
  std::vector<int32_t> e2n(2 * (E + NP));
  std::vector<double2> eS(E + NP);
  for (int64_t e = 0; e < E; ++e) {
    e2n[2 * e] = d->edge2node[2 * e];
    e2n[2 * e + 1] = d->edge2node[2 * e + 1];
    eS[e] = make_double2(d->dual_normals[2 * e], d->dual_normals[2 * e + 1]);
  }
  for (int64_t k = 0; k < NP; ++k) {
    e2n[2 * (E + k)] = d->pole_edges[2 * k];
    e2n[2 * (E + k) + 1] = d->pole_edges[2 * k + 1];
    eS[E + k] = make_double2(0.0, d->pole_normals[k]);
  }
  std::vector<double> cos_n(d->cos_lat, d->cos_lat + V);
  SweepPlan sp;
  const bool sweep_ok = nrings <= V / 4 && sweep_plan(rings_of(d), perm, tile_ptr, rowp, nbr, sp);
  if (!sweep_ok) sp = SweepPlan();
  // the sweep's cuts: longitude parts for columns too long for whole tiles;
  // bands as well where the mesh has too few tiles to fill the chip (below
  // kSweepFewTiles no built-in shape would use them)
  const int64_t nt = (int64_t)tile_ptr.size() - 1;
  const bool bands = nt >= kSweepFewTiles && nt < kSweepMinTiles;
  std::vector<std::pair<int, int>> shapes = {{1, 1}, {2, 1}, {3, 1}};
  if (bands)
    shapes = {{1, 1}, {1, 2}, {1, 3}, {1, 4}, {1, 6}, {2, 1}, {2, 2}, {3, 1}, {3, 2}};
  std::vector<std::pair<int, int>> lshapes = {{1, 1}, {2, 1}};
  if (bands)  // (thinner bands form too many gradients twice: no plan took them)
    lshapes = {{1, 1}, {1, 2}, {2, 1}, {2, 2}};
  LaplPlan lp;
  bool l2_ok = false;
  std::vector<CutPlan> cuts(sweep_ok ? shapes.size() : 0);
  std::vector<LaplCutPlan> lcuts(sweep_ok ? lshapes.size() : 0);
  if (sweep_ok) {
    const std::vector<int64_t> off = rings_of(d);
    std::vector<int32_t> ring_of(V), inv(V);
    for (size_t j = 0; j + 1 < off.size(); ++j)
      for (int64_t i = off[j]; i < off[j + 1]; ++i) ring_of[i] = (int32_t)j;
    for (int64_t p = 0; p < V; ++p) inv[perm[p]] = (int32_t)p;
    // the three plans on threads of their own (O160's upload 44 ms; one by one,
    // and with two cuts more, 55)
    const int nthr = host_threads(nt) > 1 ? 3 : 1;
    on_threads(nthr, [&](int w) {
      for (int task = w; task < 3; task += nthr) {
        if (task == 0) {
          l2_ok = lapl_plan(off, ring_of, perm, inv, tile_ptr, rowp, nbr, lp);
        } else if (task == 1) {
          for (size_t k = 0; k < cuts.size(); ++k)
            if (!cut_plan(off, ring_of, perm, tile_ptr, rowp, nbr, shapes[k].first,
                          shapes[k].second, cuts[k]))
              cuts.clear();
        } else {
          for (size_t k = 0; k < lcuts.size(); ++k)
            if (!lapl_cut_plan(off, ring_of, perm, inv, tile_ptr, rowp, nbr, lshapes[k].first,
                               lshapes[k].second, lcuts[k]))
              lcuts.clear();
        }
      }
    });
  }
  if (!l2_ok) lp = LaplPlan();
  if (cuts.empty()) lcuts.clear();
  // cos(lat) of every incidence's neighbour, so a node's row is read with
  // contiguous loads
  std::vector<double> ncos(nbr.size());
  for (size_t r = 0; r < nbr.size(); ++r) ncos[r] = d->cos_lat[(uint32_t)nbr[r] & ~kPoleBit];
  // kernels read the incidences of a node in groups of kIncPad without
  // clamping: pad every incidence array by one group
  nbr.resize(nbr.size() + kIncPad, 0);
  S.resize(S.size() + kIncPad, make_double2(0.0, 0.0));
  inc_edge.resize(inc_edge.size() + kIncPad, 0);
  ncos.resize(ncos.size() + kIncPad, 1.0);
  sp.lref.resize(sp.lref.size() + kIncPad, 1 << 16);
  if (l2_ok) lp.lref.resize(lp.lref.size() + kIncPad, 1 << 16);

  std::unique_ptr<MeshStore> m(new (std::nothrow) MeshStore());
  if (!m) return fail(ATLAS_ENOMEM, "out of host memory");
  (void)hipGetDevice(&m->device);
  m->d.V = (int32_t)V;
  m->d.E = (int32_t)E;
  m->d.npole = (int32_t)NP;
  m->d.ntiles = (int32_t)tile_ptr.size() - 1;
  m->nincid = (int64_t)nbr.size() - kIncPad;
  m->radius = d->radius;
  m->nrings = nrings;
  m->max_degree = maxdeg;
  m->allocations.reserve(8);
  for (size_t t = 0; t + 1 < tile_ptr.size(); ++t)
    m->max_tile = std::max<int64_t>(m->max_tile, tile_ptr[t + 1] - tile_ptr[t]);
  if (sweep_ok) {
    const std::vector<int64_t> off = rings_of(d);
    for (size_t j = 0; j + 1 < off.size(); ++j) m->max_run = std::max(m->max_run, off[j + 1] - off[j]);
  }
  m->d.maxdeg = maxdeg;
  m->d.mindeg = V > 0 ? mindeg : 0;
  m->d.sweep_ok = sweep_ok ? 1 : 0;
  m->d.segmax = sp.segmax;
  m->d.l2_ok = l2_ok ? 1 : 0;
  m->d.l2_fmax = lp.fmax;
  m->d.l2_gmax = lp.gmax;
  m->d.l2_pmax = lp.pmax;
  const double *vol_d = nullptr, *cos_pd = nullptr;
  std::vector<double> zeros(V, 0.0);
  std::vector<PosRec> pos(V);
  for (int64_t p = 0; p < V; ++p) {
    pos[p].node = perm[p];
    pos[p].r0 = rowp[p];
    pos[p].r1 = rowp[p + 1];
    pos[p].selfslot = sweep_ok ? sp.selfslot[p] : 0;
    pos[p].alpha = 0.0;  // derived on the device below
    pos[p].beta = 0.0;
  }
  // node coordinates by node id (remap targets and sources), and the
  // parallels of a mesh a remap can start from
  const std::vector<double> lon_n(d->lon, d->lon + V), lat_n(d->lat, d->lat + V);
  const std::vector<int64_t> rings = rings_of(d);
  std::vector<double> rlat;
  if (zipper_conforming(d, rings)) {
    rlat.resize(rings.size() - 1);
    for (size_t j = 0; j + 1 < rings.size(); ++j) rlat[j] = d->lat[rings[j]];
    m->rs.nrings = (int32_t)rlat.size();
    m->rs.ok = 1;
  }
  Upload up;
  up.add(perm, &m->d.perm);
  up.add(rowp, &m->d.rowp);
  up.add(nbr, &m->d.nbr);
  up.add(S, &m->d.S);
  up.add(inc_edge, &m->d.inc_edge);
  up.add(zeros, &m->d.alpha);
  up.add(zeros, &m->d.beta);
  up.add(cos_n, &m->d.coslat);
  up.add(tile_ptr, &m->d.tile_ptr);
  up.add(e2n, &m->d.e2n);
  up.add(eS, &m->d.eS);
  up.add(vol_p, &vol_d);
  up.add(sp.tile_seg, &m->d.tile_seg);
  up.add(sp.seg, &m->d.seg);
  up.add(sp.seg_pos, &m->d.seg_pos);
  up.add(sp.selfslot, &m->d.selfslot);
  up.add(sp.lref, &m->d.lref);
  up.add(ncos, &m->d.ncos);
  up.add(lp.tile_seg, &m->d.l2_tile_seg);
  up.add(lp.fseg, &m->d.l2_fseg);
  up.add(lp.gseg, &m->d.l2_gseg);
  up.add(lp.seg_pos, &m->d.l2_seg_pos);
  up.add(pos, &m->d.pos);
  up.add(lon_n, &m->node_lon);
  up.add(lat_n, &m->node_lat);
  if (m->rs.ok) {
    up.add(rings, &m->rs.ring_off);
    up.add(rlat, &m->rs.ring_lat);
  }
  // what only the packing below reads
  Upload tmp;
  tmp.add(cos_p, &cos_pd);
  tmp.add(lp.gnode, &m->d.l2_gnode);
  tmp.add(lp.glref, &m->d.l2_glref);
  tmp.add(lp.lref, &m->d.l2_lref);
  tmp.add(lp.lself, &m->d.l2_lself);
  void *block = nullptr;
  if ((st = up.commit(&block)) != ATLAS_OK) return st;
  m->allocations.push_back(block);
  m->bytes += up.bytes();
  if ((st = tmp.commit(&block)) != ATLAS_OK) return st;
  if ((st = derive_scales(*m, vol_d, cos_pd, d->radius)) == ATLAS_OK && l2_ok)
    st = pack_lapl_geometry(*m, (int64_t)lp.gnode.size());
  (void)hipDeviceSynchronize();
  (void)hipFree(block);
  m->d.l2_gnode = nullptr;
  m->d.l2_glref = m->d.l2_lref = m->d.l2_lself = nullptr;
  if (st != ATLAS_OK) return st;

  // The wave-specialised forms' plans and records.  They are the larger part of
  // the store beside the register-staged Laplacian's: a mesh that fits the
  // device without them goes without, on the other forms.
  Upload opt;
  m->cuts.resize(cuts.size());
  for (size_t k = 0; k < cuts.size(); ++k) {
    SweepView &v = m->cuts[k];
    opt.add(cuts[k].tile_seg, &v.tile_seg);
    opt.add(cuts[k].seg, &v.seg);
    opt.add(cuts[k].seg_pos, &v.seg_pos);
    opt.add(cuts[k].refs, &v.refs);
    v.segmax = cuts[k].segmax;
    v.pmax = cuts[k].pmax;
    v.rings = cuts[k].rings;
    v.parts = shapes[k].first;
    v.bands = shapes[k].second;
    v.ntiles = (int32_t)cuts[k].tile_seg.size() - 1;
  }
  m->lcuts.resize(lcuts.size());
  for (size_t k = 0; k < lcuts.size(); ++k) {
    LaplView &v = m->lcuts[k];
    opt.add(lcuts[k].tile_seg, &v.tile_seg);
    opt.add(lcuts[k].fseg, &v.fseg);
    opt.add(lcuts[k].gseg, &v.gseg);
    opt.add(lcuts[k].seg_pos, &v.seg_pos);
    opt.add(lcuts[k].grefs, &v.grefs);
    opt.add(lcuts[k].orefs, &v.orefs);
    v.fmax = lcuts[k].fmax;
    v.gmax = lcuts[k].gmax;
    v.pmax = lcuts[k].pmax;
    v.rings = lcuts[k].rings;
    v.parts = lshapes[k].first;
    v.bands = lshapes[k].second;
    v.ntiles = (int32_t)lcuts[k].tile_seg.size() - 1;
  }
  if (!cuts.empty()) {
    if ((st = opt.commit(&block)) == ATLAS_OK) {
      st = pack_sweep_geometry(*m);
      if (st == ATLAS_ENOMEM) {
        (void)hipFree(block);
      } else {
        m->allocations.push_back(block);
        m->bytes += opt.bytes();
      }
    }
    if (st == ATLAS_ENOMEM) {
      m->cuts.clear();
      m->lcuts.clear();
    } else if (st != ATLAS_OK) {
      return st;
    }
  }
  // the volumes stay (diagnostics)
  m->d.vol = vol_d;
  (void)hipDeviceSynchronize();
  // bytes one operator pass reads from the mesh store (column/flat forms):
  // per position perm + rowp + alpha/beta; per incidence nbr + S;
  // per node cos(lat) (div/curl)
  m->geometry_bytes = (double)V * (4 + 4 + 16) + (double)m->nincid * (4 + 16);
  *out = m.release();
  return ATLAS_OK;
}

}  // namespace atlasx
