#include "fsi_order.h"

#include <algorithm>
#include <utility>

namespace fsi {
namespace {

struct Graph {
  int n;
  std::vector<int64_t> ptr;
  std::vector<int> adj;
};

// the pattern and its transpose (entries that both hold are listed twice)
Graph symmetric_graph(int n, const std::vector<int64_t> &rowptr, const std::vector<int> &colind) {
  Graph g{n, std::vector<int64_t>(n + 1, 0), {}};
  for (int i = 0; i < n; ++i) {
    g.ptr[i + 1] += rowptr[i + 1] - rowptr[i];
    for (int64_t p = rowptr[i]; p < rowptr[i + 1]; ++p) ++g.ptr[colind[p] + 1];
  }
  for (int i = 0; i < n; ++i) g.ptr[i + 1] += g.ptr[i];
  g.adj.resize(g.ptr[n]);
  std::vector<int64_t> at(g.ptr.begin(), g.ptr.end() - 1);
  for (int i = 0; i < n; ++i)
    for (int64_t p = rowptr[i]; p < rowptr[i + 1]; ++p) {
      g.adj[at[i]++] = colind[p];
      g.adj[at[colind[p]]++] = i;
    }
  return g;
}

// distances from s into level (those of its component must be -1 before);
// returns the component's nodes by distance
std::vector<int> distances(const Graph &g, int s, std::vector<int> &level) {
  std::vector<int> order{s};
  level[s] = 0;
  for (size_t k = 0; k < order.size(); ++k) {
    const int i = order[k];
    for (int64_t p = g.ptr[i]; p < g.ptr[i + 1]; ++p)
      if (level[g.adj[p]] < 0) {
        level[g.adj[p]] = level[i] + 1;
        order.push_back(g.adj[p]);
      }
  }
  return order;
}

int smallest_degree(const Graph &g, const std::vector<int> &nodes, size_t from) {
  int best = nodes[from];
  for (size_t k = from + 1; k < nodes.size(); ++k)
    if (g.ptr[nodes[k] + 1] - g.ptr[nodes[k]] < g.ptr[best + 1] - g.ptr[best]) best = nodes[k];
  return best;
}

// first index of the nodes in the last level
size_t last_level(const std::vector<int> &nodes, const std::vector<int> &level) {
  size_t k = nodes.size();
  while (k > 0 && level[nodes[k - 1]] == level[nodes.back()]) --k;
  return k;
}

void panels(int n, const std::vector<int64_t> &rowptr, const std::vector<int> &colind, int nb, BandOrder &b) {
  std::vector<int> first(n, 0), last(n, 0), count(n + 1, 0);
  for (int i = 0; i < n; ++i) {
    if (rowptr[i] == rowptr[i + 1]) continue;
    first[i] = n;
    for (int64_t p = rowptr[i]; p < rowptr[i + 1]; ++p) {
      first[i] = std::min(first[i], b.colpos[colind[p]]);
      last[i] = std::max(last[i], b.colpos[colind[p]]);
    }
  }
  for (int i = 0; i < n; ++i) ++count[first[i] + 1];
  for (int c = 0; c < n; ++c) count[c + 1] += count[c];   // rows that begin before column c + 1
  std::vector<int> at(count.begin(), count.end() - 1);
  b.rowpos.resize(n);
  std::vector<int> lastof(n);
  for (int i = 0; i < n; ++i) {
    b.rowpos[i] = at[first[i]]++;
    lastof[b.rowpos[i]] = last[i];
  }
  const int np = (n + nb - 1) / nb;
  b.hi.resize(np);
  b.cend.resize(np);
  b.window = 0;
  int end = 0, row = 0;
  for (int p = 0; p < np; ++p) {
    b.hi[p] = count[std::min((p + 1) * nb, n)];
    for (; row < b.hi[p]; ++row) end = std::max(end, lastof[row] + 1);
    b.cend[p] = std::max(end, std::min((p + 1) * nb, n));
    b.window = std::max(b.window, b.hi[p] - p * nb);
    b.full = b.full && b.hi[p] >= std::min((p + 1) * nb, n);
  }
}

}  // namespace

BandOrder band_order(int n, const std::vector<int64_t> &rowptr, const std::vector<int> &colind, int nb) {
  const Graph g = symmetric_graph(n, rowptr, colind);
  std::vector<int> la(n, -1), lb(n, -1), seen(n, 0);
  BandOrder best;
  std::vector<int> order[2];
  for (int i = 0; i < n; ++i) {
    if (seen[i]) continue;
    // two far ends of this component: from the last level of each search on,
    // while the levels grow
    std::vector<int> nodes = distances(g, i, la);
    for (int v : nodes) seen[v] = 1;
    int start = smallest_degree(g, nodes, 0), far = start, depth = -1;
    while (true) {
      for (int v : nodes) la[v] = -1;
      nodes = distances(g, start, la);
      if (la[nodes.back()] <= depth) break;
      depth = la[nodes.back()];
      far = smallest_degree(g, nodes, last_level(nodes, la));
      std::swap(start, far);
    }
    for (int v : nodes) la[v] = -1;
    nodes = distances(g, far, la);
    (void)distances(g, start, lb);
    std::sort(nodes.begin(), nodes.end());
    for (int dir = 0; dir < 2; ++dir) {
      std::stable_sort(nodes.begin(), nodes.end(), [&](int a, int b) {
        return dir ? la[a] - lb[a] > la[b] - lb[b] : la[a] - lb[a] < la[b] - lb[b];
      });
      order[dir].insert(order[dir].end(), nodes.begin(), nodes.end());
      if (!dir) std::sort(nodes.begin(), nodes.end());
    }
  }
  for (int dir = 0; dir < 2; ++dir) {
    BandOrder b;
    b.colpos.resize(n);
    for (int k = 0; k < n; ++k) b.colpos[order[dir][k]] = k;
    panels(n, rowptr, colind, nb, b);
    const bool full = b.full;   // (singular in one direction, singular in both)
    if (!dir || b.window < best.window) best = std::move(b);
    best.full = best.full && full;
  }
  return best;
}

double band_time(const BandOrder &b, int n) {
  double rows = 0, entries = 0;
  const int np = (int)b.hi.size();
  for (int p = 0; p < np; ++p) {
    const double wait = b.hi[p] - 16 * p;
    rows += wait;
    entries += wait * std::max(b.cend[p] - std::min(16 * (p + 1), n), 0);
  }
  return 110 + 3.2 * np + 0.077 * rows + 3.2e-4 * entries;
}

double chain_time(int n) {
  return n <= 1536 ? 60 + (n + 15) / 16 * (20 + n / 60.0) : 60 + (n + 7) / 8 * (10 + n / 96.0);
}

}  // namespace fsi
