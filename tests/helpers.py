"""Small helpers shared by the CPU tests: tiny graph builders and finite differences."""
import numpy as np


def tiny_graph(n, edges):
    """edges: list of (src, dst), duplicates allowed -> CSR by destination, stable order."""
    edges = sorted(edges, key=lambda e: (e[1], e[0]))
    indptr = np.zeros(n + 1, dtype=np.int32)
    for _, d in edges:
        indptr[d + 1] += 1
    indptr = np.cumsum(indptr).astype(np.int32)
    indices = np.array([s for s, _ in edges], dtype=np.int32).reshape(-1)
    return indptr, indices


def random_graph(rng, n, m, self_loops=True, duplicates=False):
    src = rng.integers(0, n, size=m)
    dst = rng.integers(0, n, size=m)
    edges = list(zip(src.tolist(), dst.tolist()))
    if not duplicates:
        edges = list(dict.fromkeys(edges))
    if self_loops:
        edges += [(v, v) for v in range(n) if (v, v) not in set(edges)]
    return tiny_graph(n, edges)


def finite_difference(fun, theta, h=1e-6, max_entries=None, rng=None):
    """Central differences of the scalar fun at theta (fp64), entry by entry."""
    theta = np.array(theta, dtype=np.float64)
    flat = theta.reshape(-1)
    idx = np.arange(flat.size)
    if max_entries is not None and flat.size > max_entries:
        idx = rng.choice(flat.size, size=max_entries, replace=False)
    g = np.zeros(idx.size)
    for j, i in enumerate(idx):
        old = flat[i]
        flat[i] = old + h
        fp = fun(theta)
        flat[i] = old - h
        fm = fun(theta)
        flat[i] = old
        g[j] = (fp - fm) / (2 * h)
    return idx, g


# Products of fp32 operands as three bf16 parts each (six partial products): relative 2-norm error over a whole result.
# The kernels show 3e-8 (16 terms) to 4.4e-7 (233 000); without one of the partial products it is 2.4e-6 or more,
# whatever the number of terms.
PRODUCT_RTOL = 1e-6


def relative_error(got, ref):
    return np.linalg.norm(np.asarray(got, dtype=np.float64) - ref) / np.linalg.norm(ref)


def graph_with_unheard_vertices(rng, n, pairs, block_cols):
    """A random graph whose first vertex of every column block is without edges, but for one: vertex `block_cols` hears from
    vertex 3 and is heard by vertex 5.  Most rows have no multiple of four edges in a block."""
    indptr, indices = random_graph(rng, n, pairs, self_loops=False, duplicates=True)
    rows = [indices[indptr[v]:indptr[v + 1]] for v in range(n)]
    rows = [row[row % block_cols != 0] if v % block_cols else row[:0] for v, row in enumerate(rows)]
    rows[block_cols] = np.array([3])
    rows[5] = np.sort(np.append(rows[5], block_cols))
    indptr = np.concatenate(([0], np.cumsum([len(r) for r in rows]))).astype(np.int32)
    return indptr, np.concatenate(rows).astype(np.int32)


def sparse_graph_with_hubs(rng, n, hubs):
    """Rows of 0 to 3 edges, sources ascending; with hubs also rows of n and n / 2 and a vertex that every third row gathers."""
    deg = rng.integers(0, 4, n)
    if hubs:
        deg[7], deg[n - 3] = n, n // 2
    indptr = np.concatenate(([0], np.cumsum(deg))).astype(np.int32)
    row = np.repeat(np.arange(n), deg)
    src = rng.integers(0, n, len(row))
    if hubs:
        first = indptr[:-1][(deg > 0) & (np.arange(n) % 3 == 0)]
        src[first] = 11
    return indptr, src[np.lexsort((src, row))].astype(np.int32)
