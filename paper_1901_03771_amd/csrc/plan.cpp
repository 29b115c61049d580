// Materialiser and fusion partitioner.
//
// Section 2 of the paper: on a request the DAG is walked back from the
// requested node to materialised nodes; Algorithm 1 (create_subgraph) splits
// the visited sub-DAG into an ordered list of sub-graphs, cutting at nodes that
// must be materialised (materialize_node: library-grade contractions and
// reductions), at operands of such library operations
// (materialize_pred_of_node, with a transposed operand folded into the call),
// and at nodes that a second sub-graph would otherwise recompute (the
// multiple-use rule: such a node is materialised once and is a leaf of every
// user).  This file implements that rule set in closed form:
//
//   cut(n) :=  n is the requested root
//           |  n is a dot node whose consumers cannot run as its epilogue
//           |  n is the (view-stripped) lazy operand of a dot node
//           |  n is a reduction that cannot stay resident in registers
//           |  n is reached from two different cut nodes
//
// and every cut node becomes the root of one sub-graph; ascending node ids are
// a topological order, so the list is in execution order.  Two relaxations of
// the paper's rules are deliberate: a reduction over the innermost axis whose
// row fits in registers stays fused with producers and consumers, and
// pointwise consumers of a dot run as the contraction kernel's epilogue.
//
// For each sub-graph the point function of Section 3.1 is built as a flat SSA
// program: output indices are translated back to leaf indices through
// broadcast, slice and transpose nodes by composing affine per-dimension maps.
#include <algorithm>
#include <cstdio>
#include <functional>
#include <sstream>

#include "codegen.h"
#include "ctx.h"

namespace gr {

namespace {

int64_t floordiv(int64_t a, int64_t b) { int64_t q = a / b; return (a % b != 0 && ((a < 0) != (b < 0))) ? q - 1 : q; }
int64_t floormod(int64_t a, int64_t b) { return a - floordiv(a, b) * b; }

const char* op_name(int op) {
  switch (op) {
    case GR_NEG: return "neg"; case GR_ABS: return "abs"; case GR_EXP: return "exp"; case GR_LOG: return "log";
    case GR_SQRT: return "sqrt"; case GR_SQUARE: return "square"; case GR_TANH: return "tanh"; case GR_ERF: return "erf";
    case GR_ADD: return "add"; case GR_SUB: return "sub"; case GR_MUL: return "mul"; case GR_DIV: return "div";
    case GR_MAXIMUM: return "maximum"; case GR_MINIMUM: return "minimum";
    case GR_SUM: return "sum"; case GR_MAX: return "max"; case GR_MIN: return "min";
  }
  return "?";
}

std::string node_label(const Node* n) {
  switch (n->kind) {
    case Kind::LEAF: return "leaf";
    case Kind::SCALAR: return "scalar";
    case Kind::CONST: return "const";
    case Kind::UNARY: case Kind::BINARY: case Kind::REDUCE: return op_name(n->op);
    case Kind::SLICE: return "slice";
    case Kind::TRANSPOSE: return "transpose";
    case Kind::RESHAPE: return "reshape";
    case Kind::DOT: return "dot";
    case Kind::SCAN: return std::string("cum") + op_name(n->op);
  }
  return "?";
}

struct Invalid {
  const Node* node;
  std::string why;
};

// A contraction over at most eight terms (points times a 3 x 3 matrix, a handful of weights) is
// written out as products and sums inside the point function: it fuses with producers and
// consumers like any pointwise op instead of becoming a library-style kernel of its own.
bool small_dot(const Node* n) {
  return n->kind == Kind::DOT && n->ndim >= 1 && n->in[1]->shape[0] <= 8;
}

// Builds the SSA program of one sub-graph.
struct Builder {
  GroupPlan* g;
  const NodeSet* owned;  // lazy nodes this sub-graph computes
  int rank = 0;                        // iteration rank (original dims)
  const int64_t* dims = nullptr;
  std::vector<Instr>* prog = nullptr;

  std::map<std::pair<uint64_t, std::vector<int64_t>>, int> memo;
  std::map<std::vector<int64_t>, int> load_ids;   // (group, delta...) -> instr
  std::map<std::vector<int64_t>, int> value_ids;  // (kind, op, dtype, a, b) -> instr
  std::map<const Node*, int, NodeIdLess> phase_of;
  const Node* dot_core = nullptr;
  std::vector<Invalid> invalid;
  NodeSet leaves_seen, members_seen;

  static std::vector<int64_t> flatten(const IndexMap& m) {
    std::vector<int64_t> v;
    v.reserve(m.size() * 3);
    for (const DimMap& d : m) { v.push_back(d.src); v.push_back(d.scale); v.push_back(d.off); }
    return v;
  }

  void canonicalize(const Node* n, IndexMap& m) const {
    for (int d = 0; d < n->ndim; ++d) {
      DimMap& e = m[d];
      if (n->shape[d] == 1) { e = DimMap{-1, 0, 0}; continue; }
      if (e.src >= 0 && (e.scale == 0 || dims[e.src] == 1)) e = DimMap{-1, 0, e.off};
    }
  }

  int push(const Instr& in) {
    prog->push_back(in);
    return (int)prog->size() - 1;
  }

  int value_number(Instr in) {
    std::vector<int64_t> key{(int64_t)in.kind, in.op, (int64_t)in.dtype, in.a, in.b, in.cslot, in.phase};
    auto it = value_ids.find(key);
    if (it != value_ids.end()) return it->second;
    int id = push(in);
    value_ids[key] = id;
    return id;
  }

  int constant(gr_dtype dt, double v) {
    int slot = -1;
    for (size_t i = 0; i < g->consts.size(); ++i)
      if (g->consts[i].dtype == dt && std::memcmp(&g->consts[i].value, &v, sizeof(double)) == 0) slot = (int)i;
    if (slot < 0) { g->consts.push_back(ConstSlot{dt, v}); slot = (int)g->consts.size() - 1; }
    Instr in;
    in.kind = IKind::CONST; in.dtype = dt; in.cslot = slot; in.uniform = true;
    return value_number(in);
  }

  int load(const Node* leaf, const IndexMap& m) {
    leaves_seen.insert(leaf);
    std::vector<int64_t> ident{(int64_t)leaf->id};
    int64_t delta[MAXD] = {0};
    for (int d = 0; d < leaf->ndim; ++d) {
      const DimMap& e = m[d];
      ident.push_back(e.src);
      ident.push_back(e.scale);
      if (e.src < 0) ident.push_back(e.off);
      else { ident.push_back(floormod(e.off, e.scale)); delta[e.src] += floordiv(e.off, e.scale); }
    }
    int gid = -1;
    for (size_t i = 0; i < g->groups.size(); ++i) if (g->groups[i].ident == ident) gid = (int)i;
    if (gid < 0) {
      AccessGroup ag;
      ag.leaf = leaf; ag.dtype = leaf->dtype; ag.ident = ident;
      ag.base = leaf->offset;
      for (int k = 0; k < MAXD; ++k) ag.structural_zero[k] = true;
      for (int d = 0; d < leaf->ndim; ++d) {
        const DimMap& e = m[d];
        if (e.src < 0) ag.base += leaf->strides[d] * e.off;
        else {
          ag.base += leaf->strides[d] * floormod(e.off, e.scale);
          ag.coef[e.src] += leaf->strides[d] * e.scale;
          ag.structural_zero[e.src] = false;
        }
      }
      g->groups.push_back(ag);
      gid = (int)g->groups.size() - 1;
    }
    std::vector<int64_t> dv(delta, delta + rank);
    g->groups[gid].deltas.insert(dv);
    std::vector<int64_t> key{gid};
    key.insert(key.end(), dv.begin(), dv.end());
    auto it = load_ids.find(key);
    if (it != load_ids.end()) return it->second;
    Instr in;
    in.kind = IKind::LOAD; in.dtype = leaf->dtype; in.group = gid;
    for (int k = 0; k < rank; ++k) in.delta[k] = delta[k];
    in.uniform = g->groups[gid].structural_zero[rank - 1];
    int id = push(in);
    load_ids[key] = id;
    return id;
  }

  static bool is_identity_on(const IndexMap& m, int d, int src, int64_t extent) {
    if (extent == 1) return true;  // canonicalised to a constant 0
    return m[d].src == src && m[d].scale == 1 && m[d].off == 0;
  }

  int eval(const Node* n, IndexMap m) {
    canonicalize(n, m);
    auto key = std::make_pair(n->id, flatten(m));
    auto it = memo.find(key);
    if (it != memo.end()) return it->second;
    int id = -1;
    if (n->kind == Kind::CONST) {
      id = constant(n->dtype, n->value);
    } else if (n->has_data()) {
      id = load(n, m);
    } else {
      members_seen.insert(n);
      switch (n->kind) {
        case Kind::UNARY: {
          Instr in;
          in.kind = IKind::UNARY; in.op = n->op; in.dtype = n->dtype;
          in.a = eval(n->in[0], m);
          in.uniform = (*prog)[in.a].uniform;
          id = value_number(in);
          break;
        }
        case Kind::BINARY: {
          int ops[2];
          for (int s = 0; s < 2; ++s) {
            const Node* o = n->in[s];
            IndexMap om(o->ndim);
            for (int d = 0; d < o->ndim; ++d) om[d] = m[d + (n->ndim - o->ndim)];
            ops[s] = eval(o, om);  // canonicalize() zeroes broadcast (extent-1) dims
          }
          Instr in;
          in.kind = IKind::BINARY; in.op = n->op; in.dtype = n->dtype; in.a = ops[0]; in.b = ops[1];
          in.uniform = (*prog)[in.a].uniform && (*prog)[in.b].uniform;
          id = value_number(in);
          break;
        }
        case Kind::SLICE: {
          IndexMap om(n->ndim);
          for (int d = 0; d < n->ndim; ++d)
            om[d] = DimMap{m[d].src, m[d].scale * n->step[d], n->start[d] + n->step[d] * m[d].off};
          id = eval(n->in[0], om);
          break;
        }
        case Kind::TRANSPOSE: {
          IndexMap om(n->ndim);
          for (int d = 0; d < n->ndim; ++d) om[n->perm[d]] = m[d];
          id = eval(n->in[0], om);
          break;
        }
        case Kind::REDUCE: {
          id = reduce_result(n, m);
          break;
        }
        case Kind::DOT: {
          if (small_dot(n)) {
            const Node* A = n->in[0];
            const Node* B = n->in[1];
            const int64_t K = B->shape[0];
            // the sum starts from +0 like the accumulator of a contraction kernel (and of the eager
            // evaluation): products that are all -0 add up to +0
            id = constant(n->dtype, 0.0);
            for (int64_t k = 0; k < K; ++k) {
              IndexMap am(A->ndim), bm(B->ndim);
              if (A->ndim == 2) am[0] = m[0];
              am[A->ndim - 1] = DimMap{-1, 0, k};
              bm[0] = DimMap{-1, 0, k};
              if (B->ndim == 2) bm[1] = m[n->ndim - 1];
              Instr mul;
              mul.kind = IKind::BINARY; mul.op = GR_MUL; mul.dtype = n->dtype;
              mul.a = eval(A, am); mul.b = eval(B, bm);
              mul.uniform = (*prog)[mul.a].uniform && (*prog)[mul.b].uniform;
              int p = value_number(mul);
              Instr add;
              add.kind = IKind::BINARY; add.op = GR_ADD; add.dtype = n->dtype; add.a = id; add.b = p;
              add.uniform = (*prog)[id].uniform && (*prog)[p].uniform;
              id = value_number(add);
            }
            break;  // (an empty contraction is the constant 0)
          }
          bool ok = (g->kind == GroupKind::GEMV || g->kind == GroupKind::GEMM) && (dot_core == nullptr || dot_core == n);
          for (int d = 0; ok && d < n->ndim; ++d) ok = is_identity_on(m, d, d, n->shape[d]);
          if (!ok) { invalid.push_back({n, "dot result not usable as an epilogue input"}); id = constant(GR_F32, 0.0); break; }
          dot_core = n;
          Instr in;
          in.kind = IKind::ACC; in.dtype = GR_F32;
          id = value_number(in);
          break;
        }
        case Kind::SCAN:
          invalid.push_back({n, "a scan is always materialised"});
          id = constant(n->dtype, 0.0);
          break;
        default:
          invalid.push_back({n, "unexpected lazy node kind (" + node_label(n) + " #" + std::to_string(n->id) + ")"});
          id = constant(GR_F32, 0.0);
      }
    }
    memo[key] = id;
    return id;
  }

  // A reduction met inside a row-resident sub-graph: its value for the current
  // row is the result of one reduction phase over the row.
  int reduce_result(const Node* r, const IndexMap& m) {
    const Node* x = r->in[0];
    bool ok = g->kind == GroupKind::ROWRED && x->ndim == rank && x->ndim >= 1;
    if (ok) for (int d = 0; d < x->ndim; ++d) {
      if (r->red_axis[d] != (d == x->ndim - 1)) ok = false;
      if (x->shape[d] != dims[d]) ok = false;
    }
    if (ok) {
      int kept = x->ndim - 1;
      if ((int)m.size() != (r->keepdims ? x->ndim : kept)) ok = false;
      for (int d = 0; ok && d < kept; ++d) if (!is_identity_on(m, d, d, x->shape[d])) ok = false;
    }
    if (!ok) {
      invalid.push_back({r, "reduction cannot stay row-resident in this sub-graph"});
      return constant(r->dtype, 0.0);
    }
    auto it = phase_of.find(r);
    int ph;
    if (it != phase_of.end()) ph = it->second;
    else {
      IndexMap full(x->ndim);
      for (int d = 0; d < x->ndim; ++d) full[d] = DimMap{d, 1, 0};
      int v = eval(x, full);
      Phase p;
      p.op = r->op; p.in_dtype = x->dtype; p.out_dtype = r->dtype; p.value = v; p.node = r;
      g->phases.push_back(p);
      ph = (int)g->phases.size() - 1;
      phase_of[r] = ph;
    }
    Instr in;
    in.kind = IKind::RED; in.dtype = r->dtype; in.phase = ph; in.uniform = true;
    return value_number(in);
  }
};

// Follows views from `n` down to a node with data, composing the index map.
bool resolve_to_leaf(const Node* n, IndexMap m, const Node** leaf, IndexMap* lm) {
  while (!n->has_data()) {
    if (n->kind == Kind::SLICE) {
      IndexMap om(n->ndim);
      for (int d = 0; d < n->ndim; ++d) om[d] = DimMap{m[d].src, m[d].scale * n->step[d], n->start[d] + n->step[d] * m[d].off};
      m = om;
    } else if (n->kind == Kind::TRANSPOSE) {
      IndexMap om(n->ndim);
      for (int d = 0; d < n->ndim; ++d) om[n->perm[d]] = m[d];
      m = om;
    } else return false;
    n = n->in[0];
  }
  *leaf = n;
  *lm = m;
  return true;
}

// A contraction with one output row or very few, over a long k: too little parallelism for the
// row-per-lane-group kernel.  It is planned as the map-reduce it is (Listing 5 of the paper writes
// the inner product exactly so): value a[m,k] * v[k], reduced over k in two stages.
// Element strides an array will have when it is read: those of its storage if it has one, of a
// C-contiguous result if it is still to be computed, transformed by the views in between.
static void strides_when_read(const Node* n, int64_t* st) {
  if (n->materialized) { for (int d = 0; d < n->ndim; ++d) st[d] = n->strides[d]; return; }
  if (!n->is_view()) {
    int64_t s = 1;
    for (int d = n->ndim - 1; d >= 0; --d) { st[d] = s; s *= n->shape[d]; }
    return;
  }
  int64_t in[MAXD];
  strides_when_read(n->in[0], in);
  if (n->kind == Kind::SLICE) for (int d = 0; d < n->ndim; ++d) st[d] = in[d] * n->step[d];
  else for (int d = 0; d < n->ndim; ++d) st[d] = in[n->perm[d]];
}

bool dot_as_reduce(const Node* n) {
  if (n->kind != Kind::DOT) return false;
  const Node* A = n->in[0];
  const Node* v = n->in[1];
  if (v->ndim != 1) return false;
  const int64_t K = v->shape[0], M = A->ndim == 2 ? A->shape[0] : 1;
  if (!(K >= 8192 && M * 64 <= K && M <= 2048)) return false;
  // rows that are contiguous along k only: a transposed matrix has the column-accumulate kernel
  int64_t st[MAXD];
  strides_when_read(A, st);
  return st[A->ndim - 1] == 1 || st[A->ndim - 1] == 2 || A->ndim == 1;
}

// The node whose index space a map sub-graph rooted at `r` iterates over: the operand of a reshape
// that is still to be evaluated, `r` itself otherwise.
const Node* map_source(const Node* r) {
  return (r->kind == Kind::RESHAPE && !r->materialized && !r->in.empty()) ? r->in[0] : r;
}

const Node* strip_views(const Node* n) {
  while (n->is_view() && !n->has_data()) n = n->in[0];
  return n;
}

int next_pow2(int64_t v) { int p = 1; while (p < v && p < (1 << 30)) p <<= 1; return p; }  // saturates at 2^30

void normalize_deltas(GroupPlan* g, std::vector<Instr>* progs[], int nprogs, int rank) {
  for (size_t gi = 0; gi < g->groups.size(); ++gi) {
    AccessGroup& ag = g->groups[gi];
    if (ag.deltas.empty()) continue;
    std::vector<int64_t> mn(rank, INT64_MAX);
    for (const auto& d : ag.deltas) for (int k = 0; k < rank; ++k) mn[k] = std::min(mn[k], d[k]);
    std::set<std::vector<int64_t>> nd;
    for (auto d : ag.deltas) { for (int k = 0; k < rank; ++k) d[k] -= mn[k]; nd.insert(d); }
    ag.deltas.swap(nd);
    for (int k = 0; k < rank; ++k) ag.base += ag.coef[k] * mn[k];
    for (int p = 0; p < nprogs; ++p)
      for (Instr& in : *progs[p])
        if (in.kind == IKind::LOAD && in.group == (int)gi) for (int k = 0; k < rank; ++k) in.delta[k] -= mn[k];
  }
}

// Merges adjacent iteration dimensions that every access (and the contiguous
// output) walks as one linear run.  `barrier[k]` forbids merging dim k with k+1.
void collapse_dims(GroupPlan* g, const bool* barrier, std::vector<Instr>* progs[], int nprogs) {
  int n = g->orig_rank;
  // runs of original dims, extent-1 dims dropped
  std::vector<std::vector<int>> runs;
  for (int k = 0; k < n; ++k) {
    if (g->orig_dims[k] == 1) continue;
    bool merged = false;
    if (!runs.empty()) {
      int prev = runs.back().back();
      bool blocked = false;
      for (int j = prev; j < k; ++j) if (barrier[j]) blocked = true;
      if (!blocked) {
        // prev (outer) merges with k (inner) if coef[prev] == coef[k] * dims[k] everywhere,
        // and no access is shifted in the outer dim
        bool ok = true;
        for (const AccessGroup& ag : g->groups) {
          if (ag.coef[prev] != ag.coef[k] * g->orig_dims[k]) ok = false;
          for (const auto& d : ag.deltas) if (d[prev] != 0) ok = false;
        }
        if (ok) { runs.back().push_back(k); merged = true; }
      }
    }
    if (!merged) runs.push_back({k});
  }
  if (runs.empty()) runs.push_back({n - 1});
  // a run (outer..inner) was built by appending inner dims; verify pairwise chain (outer vs next) held
  g->rank = (int)runs.size();
  for (int k = 0; k < MAXD; ++k) g->collapse_to[k] = -1;
  for (int r = 0; r < g->rank; ++r) {
    int64_t e = 1;
    for (int k : runs[r]) { e *= g->orig_dims[k]; g->collapse_to[k] = r; }
    g->dims[r] = e;
  }
  for (AccessGroup& ag : g->groups) {
    int64_t nc[MAXD] = {0};
    bool nz[MAXD];
    for (int r = 0; r < g->rank; ++r) { nc[r] = ag.coef[runs[r].back()]; nz[r] = ag.structural_zero[runs[r].back()]; }
    std::set<std::vector<int64_t>> nd;
    for (const auto& d : ag.deltas) {
      std::vector<int64_t> v(g->rank);
      for (int r = 0; r < g->rank; ++r) v[r] = d[runs[r].back()];
      nd.insert(v);
    }
    ag.deltas.swap(nd);
    for (int r = 0; r < MAXD; ++r) { ag.coef[r] = r < g->rank ? nc[r] : 0; ag.structural_zero[r] = r < g->rank ? nz[r] : true; }
  }
  for (int p = 0; p < nprogs; ++p)
    for (Instr& in : *progs[p])
      if (in.kind == IKind::LOAD) {
        int64_t v[MAXD] = {0};
        for (int r = 0; r < g->rank; ++r) v[r] = in.delta[runs[r].back()];
        for (int r = 0; r < MAXD; ++r) in.delta[r] = v[r];
      }
}

void put(std::string& s, int64_t v) { s.append(reinterpret_cast<const char*>(&v), sizeof(v)); }

void dump_prog(std::string& s, const std::vector<Instr>& prog, int rank) {
  for (const Instr& in : prog) {
    put(s, ((int64_t)in.kind << 48) | ((int64_t)in.op << 32) | ((int64_t)in.dtype << 16) | (int64_t)in.uniform);
    put(s, ((int64_t)(in.a + 1) << 32) | (int64_t)(in.b + 1));
    put(s, ((int64_t)(in.group + 1) << 40) | ((int64_t)(in.cslot + 1) << 20) | (int64_t)(in.phase + 1));
    if (in.kind == IKind::LOAD) for (int k = 0; k < rank; ++k) put(s, in.delta[k]);
  }
}

// Cache key: everything the generated source depends on, and nothing else (extents,
// strides, base offsets and constants are kernel arguments).
void make_signature(GroupPlan* g) {
  std::string s;
  s.reserve(256 + 32 * (g->prog.size() + g->prog1.size()));
  for (int64_t v : {(int64_t)g->kind, (int64_t)g->rank, (int64_t)g->out_dtype, (int64_t)g->out_per_row, (int64_t)g->BX, (int64_t)g->BY,
                    (int64_t)g->VR + (g->kind == GroupKind::GEMM && g->VR == 2 && g->slabs > 1 ? 1024 : 0) /* (the direct-to-LDS product kernels compile the split of K in or out) */, (int64_t)g->UC, (int64_t)g->NP, (int64_t)g->row_threads + 1024 * (int64_t)g->row_iters + (((int64_t)g->pair_k) << 32) + (((int64_t)g->pair_lane) << 40) /* (a pair kernel compiles its row length in) */, (int64_t)g->xcd_remap + 2 * (int64_t)g->stage_mask + (((int64_t)g->tail) << 40) + (((int64_t)g->diag) << 44) + (((int64_t)g->cphase) << 48) + (((int64_t)g->flat) << 52) + (((int64_t)g->in_place) << 56) + (((int64_t)g->in_place_once) << 57), (int64_t)g->red_mode + 16 * (int64_t)g->red_vec,
                    (int64_t)g->red_kept_rank, (int64_t)g->gemv_mode, (int64_t)g->LPR, (int64_t)g->KV, (int64_t)g->mat_group,
                    (int64_t)g->vec_group, (int64_t)g->nt, (int64_t)g->unroll, (int64_t)g->scan_mode + 16 * (int64_t)g->scan_vec + (g->scan_mode >= 2 ? 256 * g->scan_chunk : 0) /* (a one-pass scan's tile size is compiled in) */, (int64_t)g->out_unit, (int64_t)g->groups.size()})
    put(s, v);
  for (const AccessGroup& ag : g->groups) {
    int64_t cls = (int64_t)ag.dtype;
    bool core = g->kind == GroupKind::GEMV;
    int nd = core ? 2 : g->rank;
    for (int k = 0; k < nd; ++k) cls = cls * 4 + (ag.structural_zero[k] ? 0 : (ag.coef[k] == 1 ? 1 : 2));
    put(s, cls);
  }
  if (g->in_place) put(s, (int64_t)g->self_row * 256 + g->self_col);
  put(s, (int64_t)g->consts.size());
  for (const ConstSlot& c : g->consts) put(s, (int64_t)c.dtype);
  put(s, (int64_t)g->phases.size());
  for (const Phase& p : g->phases) put(s, ((int64_t)p.op << 40) | ((int64_t)p.in_dtype << 32) | ((int64_t)p.out_dtype << 24) | (int64_t)p.value);
  put(s, (int64_t)g->results.size());
  if (g->kind != GroupKind::MAP) { for (int r : g->results) put(s, r); dump_prog(s, g->prog, g->rank); }
  put(s, g->result1);
  dump_prog(s, g->prog1, g->rank);
  if (g->pair) { s.append("|pair|"); s.append(g->pair->signature); }
  g->signature.swap(s);
}

// The output takes part in dimension collapsing as one more access (its strides need not be
// those of a C-contiguous array when the root is written through a slice assignment).
void push_output_group(GroupPlan* g, int n) {
  AccessGroup og;
  og.leaf = nullptr;
  og.dtype = g->out_dtype;
  for (int k = 0; k < MAXD; ++k) og.structural_zero[k] = true;
  for (int k = 0; k < n; ++k) { og.coef[k] = g->out_orig_coef[k]; og.structural_zero[k] = g->orig_dims[k] == 1; }
  og.deltas.insert(std::vector<int64_t>(n, 0));
  g->groups.push_back(og);
}

void pop_output_group(GroupPlan* g) {
  for (int k = 0; k < g->rank; ++k) g->out_coef[k] = g->groups.back().coef[k];
  g->groups.pop_back();
  g->out_unit = g->out_coef[g->rank - 1] == 1 || g->dims[g->rank - 1] == 1;
}

struct Planner {
  gr_ctx* c;
  Node* root;
  const OutSpec* out = nullptr;
  std::vector<Node*> sub;                 // lazy nodes of the visited sub-DAG, ascending id
  NodeSet cuts;
  std::map<const Node*, const Node*, NodeIdLess> owner;

  void collect() {
    std::set<Node*> seen;
    std::vector<Node*> work{root};
    while (!work.empty()) {
      Node* n = work.back();
      work.pop_back();
      if (n->materialized || seen.count(n)) continue;  // a materialised node ends the walk (Section 2)
      seen.insert(n);
      for (Node* p : n->in) work.push_back(p);
    }
    sub.assign(seen.begin(), seen.end());
    std::sort(sub.begin(), sub.end(), [](Node* a, Node* b) { return a->id < b->id; });
  }

  void initial_cuts() {
    cuts.insert(root);
    for (Node* n : sub) {
      if (!c->opt_fusion && n->is_compute()) cuts.insert(n);
      if (n->kind == Kind::DOT && !small_dot(n)) {
        // operands of a contraction are materialised first; views (a transposed
        // matrix in particular) are folded into the contraction kernel instead
        for (Node* o : n->in) {
          const Node* b = strip_views(o);
          if (!b->materialized) cuts.insert(b);
        }
      }
      if (dot_as_reduce(n)) cuts.insert(n);       // evaluated as a two-stage reduction: consumers read its result
      if (n->kind == Kind::SCAN) cuts.insert(n);  // a scan is materialised (materialize_node, Section 2)
      if (n->kind == Kind::RESHAPE) cuts.insert(n);  // a reshape is a stored copy: its consumers index it under the new shape
      if (n->kind == Kind::REDUCE) {
        const Node* x = n->in[0];
        bool last_only = x->ndim >= 1;
        for (int d = 0; d < x->ndim; ++d) if (n->red_axis[d] != (d == x->ndim - 1)) last_only = false;
        if (!last_only || x->shape[x->ndim - 1] > std::min<int64_t>(c->opt_rowred_max_cols, 65536)) cuts.insert(n);   // (64 elements of each of 1024 lanes)
      }
    }
  }

  // Returns false (after adding a cut) if some node is reached from two roots.
  bool assign_owners() {
    owner.clear();
    for (Node* r : sub) {
      if (!cuts.count(r)) continue;
      std::vector<const Node*> work;
      NodeSet seen;
      for (Node* p : r->in) work.push_back(p);
      owner[r] = r;
      while (!work.empty()) {
        const Node* n = work.back();
        work.pop_back();
        if (n->materialized || cuts.count(n) || seen.count(n)) continue;
        seen.insert(n);
        if (n->is_compute()) {
          auto it = owner.find(n);
          if (it != owner.end() && it->second != r) { cuts.insert(n); return false; }  // multiple-use rule
          owner[n] = r;
        }
        for (Node* p : n->in) work.push_back(p);
      }
    }
    return true;
  }

  NodeSet owned_by(const Node* r) const {
    NodeSet s;
    for (const auto& kv : owner) if (kv.second == r) s.insert(kv.first);
    return s;
  }
};

void choose_map_schedule(gr_ctx* c, GroupPlan* g, bool own_output) {
  int64_t C = g->dims[g->rank - 1];
  int64_t R = g->rank >= 2 ? g->dims[g->rank - 2] : 1;
  int64_t outer = 1;
  for (int k = 0; k + 2 < g->rank; ++k) outer *= g->dims[k];
  g->BX = std::min(256, std::max(1, next_pow2((C + 3) / 4)));
  if (c->opt_map_bx > 0 && c->opt_map_bx <= 256 && (c->opt_map_bx & (c->opt_map_bx - 1)) == 0) g->BX = std::min<int>(g->BX, (int)c->opt_map_bx);
  bool shifted_rows = false;
  for (const AccessGroup& ag : g->groups)
    for (const auto& d : ag.deltas) if (g->rank >= 2 && d[g->rank - 2] != 0) shifted_rows = true;
  // Programs without row-shifted views (pointwise and broadcast): a wave per 256 columns and the
  // four waves of a workgroup on neighbouring row pairs, two rows per lane (measured on MI355X,
  // normalize 8192^2: 83.0 us against 85.3 with 1024 columns by four rows per workgroup; stencils
  // keep the wide tile, 96 us against 97-113)
  // Only where every row piece of 256 columns is a run of whole 256-byte blocks in every array
  // (rows of 1024 columns or more in multiples of 256, no views shifted along the columns, row
  // strides in multiples of 64 elements): a narrow tile leaves the ends of unaligned pieces to
  // other workgroups, and their partial lines cost more than the tile shape gains (x*row on
  // 8192 x 8190: 113 us narrow, 95 us wide).
  bool aligned = C >= 1024 && C % 256 == 0;
  for (const AccessGroup& ag : g->groups) {
    if (ag.structural_zero[g->rank - 1]) continue;
    if (ag.deltas.size() != 1 || ag.coef[g->rank - 1] != 1 || ag.base % 64 != 0) aligned = false;
    for (const auto& d : ag.deltas) if (d[g->rank - 1] != 0) aligned = false;
    for (int k = 0; k + 1 < g->rank; ++k) if (!ag.structural_zero[k] && ag.coef[k] % 64 != 0) aligned = false;
  }
  for (int k = 0; k + 1 < g->rank; ++k) if (g->out_coef[k] % 64 != 0) aligned = false;
  if (g->out_base % 64 != 0) aligned = false;
  const bool narrow_tile = g->rank >= 2 && R > 1 && !shifted_rows && aligned && c->opt_map_bx == 0 && g->BX > 64;
  if (narrow_tile) g->BX = 64;
  // Views shifted by at most one row up and down (a five-point sweep): 512 columns by four rows per workgroup, two
  // rows per lane (measured on MI355X against 1024 columns by four rows with four rows per lane, right-hand side of a
  // Jacobi sweep: 8192^2 92.5 against 97.6 us, 16384 x 4096 93.5 against 104.2, 4096 x 16384 92.6 against 96.8,
  // 4096^2 30.4 against 31.2, 8190^2 90.9 against 91.7; taller stencils keep the wide tile, within 1-3 % either way)
  int64_t row_lo = 0, row_hi = 0;
  for (const AccessGroup& ag : g->groups)
    for (const auto& d : ag.deltas) if (g->rank >= 2) { row_lo = std::min(row_lo, d[g->rank - 2]); row_hi = std::max(row_hi, d[g->rank - 2]); }
  const bool low_stencil = shifted_rows && row_hi - row_lo <= 2 && c->opt_map_bx == 0 && g->BX == 256;
  if (low_stencil) g->BX = 128;
  g->BY = 256 / g->BX;
  auto tiles = [&](int vr, int uc) {
    int64_t tc = (int64_t)g->BX * 4 * uc, tr = (int64_t)g->BY * vr;
    return outer * ((C + tc - 1) / tc) * ((R + tr - 1) / tr);
  };
  g->VR = 1; g->UC = 1;
  if (g->rank == 1 || R == 1) {
    for (int uc : {4, 2}) if (tiles(1, uc) >= 2048) { g->UC = uc; break; }
  } else {
    int want = narrow_tile || low_stencil ? 2 : 4;  // measured on MI355X: 4 rows per lane is the best patch for tall stencil programs and for broadcast programs on wide tiles
    // (lanes whose patch sticks out of the array take the guarded point-by-point path: with few
    // rows the patch height has to divide them)
    for (int vr = want; vr >= 2; vr >>= 1)
      if ((R % vr == 0 || R >= 16 * vr) && (tiles(vr, 1) >= 1024 || (shifted_rows && tiles(vr, 1) >= 256))) { g->VR = vr; break; }
  }
  // Operands whose contiguous dimension is the row dimension of the iteration space (transposed
  // views): lanes along the columns would read them with a stride.  A tile (64 columns by 64 or 128 rows) of such an
  // operand is loaded along its own contiguous dimension into LDS and read from there transposed.
  g->stage_mask = 0;
  g->diag = 0;
  if (g->rank >= 2 && R >= 64 && C >= 64 && c->opt_map_rows == 0 && c->opt_map_chunks == 0 && c->opt_map_bx == 0 && c->opt_stage) {
    int staged = 0;
    for (size_t gi = 0; gi < g->groups.size() && gi < 24; ++gi) {
      const AccessGroup& ag = g->groups[gi];
      if (ag.dtype == GR_I64 || ag.deltas.size() != 1) continue;
      if (ag.structural_zero[g->rank - 1] || ag.structural_zero[g->rank - 2]) continue;
      if (ag.coef[g->rank - 1] != 1 && ag.coef[g->rank - 2] == 1 && staged < 2) { g->stage_mask |= 1 << gi; ++staged; }
    }
    // (64 columns by 64 or 128 rows: the taller tile reads 512-byte runs of the operand)
    if (g->stage_mask) { g->BX = 16; g->BY = 16; g->VR = (R >= 128 && c->opt_stage_rows != 64) ? 8 : 4; g->UC = 1; g->diag = c->opt_stage_diag != 0; }
    // Such a tile writes 256-byte pieces of output rows.  Where rows do not start on 64-byte
    // boundaries the pieces of neighbouring tiles share cache lines, which only plain stores let
    // the L2 merge (measured, 8191^2 transposed: 144 us plain, 177 us with hinted stores).
    if (g->stage_mask && (g->nt & 8) && c->opt_nontemporal == 1 && (C % 16 != 0 || g->out_coef[g->rank - 2] % 16 != 0)) g->nt &= ~8;
  }
  if (c->opt_map_rows > 0 && g->rank >= 2) g->VR = (int)std::min<int64_t>(c->opt_map_rows, 16);
  if (c->opt_map_chunks > 0) g->UC = (int)std::min<int64_t>(c->opt_map_chunks, 8);
  g->xcd_remap = shifted_rows;
  // A strided destination (the box of a slice assignment, a stencil sweep writing the interior of a
  // grid) may start off a 16-byte boundary while its rows are 16-byte multiples apart: lanes then own
  // the column groups that are aligned in the OUTPUT (the first and the last group of a row are
  // partial and take the guarded path), so that a wave's vector stores cover whole cache lines.
  g->cphase = 0;
  if (g->rank >= 2 && C >= 256 && g->out_unit && g->out_dtype != GR_I64 && !g->stage_mask && g->UC == 1 && c->opt_map_phase) {
    bool rows_aligned = true;
    for (int k = 0; k + 1 < g->rank; ++k) if (g->out_coef[k] % 4 != 0) rows_aligned = false;
    if (rows_aligned) g->cphase = (int)(((g->out_base % 4) + 4) % 4);
  }
  // Narrow arrays (points, pixels: a few columns): the lanes that own the last, incomplete group
  // of four columns are a large share of all lanes (all of them below four columns).  The kernel
  // is specialised on columns mod 4 and gives those lanes straight-line code as well.
  // Rows that are no multiple of four: the last group of columns starts four from the row's end (the last rows of a tile
  // VR from the array's), overlapping the group before it with the same values, and no lane needs the guarded path, whose
  // serial scalar loads its whole wave waits for (x * row + 1 on 300000 x 90: 58.9 -> 41.0 us, 192105 x 131: 64.1 -> 39.5,
  // 5033164 x 5: 92.6 -> 55.2, 8190^2: 95.3 -> 93.5).  Not for the destination of a slice assignment, which the value may read:
  // an element computed twice would see its own result.
  // Rows a little longer than a tile of 1024 columns leave most of the second tile's lanes idle: there the lanes are
  // numbered over all groups of four columns instead (24480 x 1028: 53.5 -> 40.3 us, 16777 x 1500: 46.7 -> 38.9; from 85 % of
  // lanes in use on and in narrower tiles the idle lanes cost less than the index arithmetic: 8388 x 3000 37.8 against
  // 38.7, 74017 x 340 36.3 against 40.5), unless the program is long enough for the idle lanes' issue slots to count
  // (division and square root per element on 100003 x 257, 65 of 128 lanes: 43 -> 35 us).  Such lanes share cache lines across waves, so their loads carry no hint.
  if (own_output && !narrow_tile && g->rank >= 2 && R > 1 && C >= 4 && g->UC == 1 && !g->stage_mask && !g->cphase && g->out_unit &&
      c->opt_map_rows == 0 && c->opt_map_chunks == 0 && c->opt_map_bx == 0) {
    const int64_t tc = (int64_t)g->BX * 4, padded = (C + tc - 1) / tc * tc;
    int64_t ops = 0;   // per element, in simple operations
    for (const Instr& in : g->prog1)
      if (!in.uniform && (in.kind == IKind::UNARY || in.kind == IKind::BINARY)) ops += heavy_op(in) ? 8 : 1;
    const bool heavy = ops >= 16 && C * 100 < padded * 80;
    if (heavy || (g->BX >= 128 && C > tc && C * 100 < padded * 85)) {
      g->flat = 1;
      g->BX = 256; g->BY = 1; g->VR = 1;
      if (c->opt_nontemporal == 1) g->nt &= ~7;
      for (int vr = 4; vr >= 2; vr >>= 1)
        if ((R % vr == 0 || R >= 16 * vr) && outer * ((C + 3) / 4) * ((R + vr - 1) / vr) >= 256 * (shifted_rows ? 256 : 1024)) { g->VR = vr; break; }
    } else if (C % 4 != 0) g->flat = 2;
  }
  // (rows shorter than 256 bytes share cache lines with other waves as well: 3145728 x 8 52.6 -> 42.6 us without the hint)
  if (c->opt_nontemporal == 1 && g->rank >= 2 && R > 1 && C < 64) g->nt &= ~7;
  g->tail = (g->rank >= 2 && !g->flat && C < 64 && (C & 3) && g->UC == 1 && !g->stage_mask) ? (int)(C & 3) : 0;
}

// Tiles up to which such a map is one launch: two per compute unit, which are all there at the same time, so that a tile that looks at the marks around its
// own finds them.  (Ten sweeps, us, two launches / one, Jacobi's five points and values four rows and columns away: 252 tiles of 1000^2 72 / 68 and 81 / 57, 284
// of 4535 x 400 101 / 88 and 104 / 82, 376 of 1500 x 1900 109 / 104 and 121 / 103, 456 of 1800^2 113 / 111 and 119 / 104, 512 of 2040^2 116 / 116.5 and 134 / 110; 576
// of 4600 x 1020 129.5 / 136 and 168 / 160, 594 of 2100^2 126 / 139 and 166 / 190, 648 of 2300^2 129 / 142 and 168 / 230, 768 of 1000 x 6000 129.5 / 149 and 177 / 338,
// 2176 of 4096^2 279 / 369.)
constexpr int64_t kOnceTiles = 512;

// A map that is to write the array it reads at shifted positions, element (r, c) from elements a few rows and columns
// away (a sweep of a stencil over a grid with a single buffer): every array read is a scalar or lies over the output with its strides.
// Tiles of 256 columns (the narrowest power of two that holds shorter rows) by eight rows per lane: taller patches save and
// read fewer rows around them, and their registers leave fewer waves (4096^2, us per sweep by 256 columns: 4 rows 28.7, 8 27.9, 16 29.7; by
// 1024: 37.0, 31.2, 29.0, of 32 rows 36.0; 8192^2 by 256, 512 and 1024 columns, 8 rows: 102, 107, 115).  Four rows where eight
// would leave compute units without a tile (1000^2: 7.8 against 8.5).
// (us per sweep, value in a buffer of its own and copied back / in place: 1000^2 9.1 / 7.8, 2000^2 20.0 / 11.8, 4096 x 1024 23.1 / 11.8,
// 100000 x 130 34.8 / 20.5, 4096^2 49.6 / 27.9, 1024 x 16384 49.1 / 26.9, 8192^2 185 / 102; both with two launches.)
static void choose_in_place(gr_ctx* c, GroupPlan* g) {
  if (g->rank != 2 || g->orig_rank != 2 || !g->out_unit || g->out_dtype == GR_I64 || g->stage_mask) return;
  const int64_t R = g->dims[0], C = g->dims[1], row = g->out_coef[0];
  if (C < 16 || R < 2 || row < C || R > 1 << 30 || C > 1 << 30) return;
  const AccessGroup* self = nullptr;
  for (const AccessGroup& ag : g->groups) {
    if (ag.structural_zero[0] && ag.structural_zero[1]) continue;
    if (self || ag.leaf->ndim != 2 || ag.dtype != g->out_dtype || ag.coef[0] != row || ag.coef[1] != 1) return;
    self = &ag;
  }
  if (!self) return;
  const int64_t d = self->base - g->out_base, dr = d >= 0 ? (d + row / 2) / row : -((row / 2 - d) / row), dc = d - dr * row;
  int64_t lo[2] = {0, 0}, hi[2] = {0, 0};
  for (const auto& s : self->deltas) {
    lo[0] = std::min(lo[0], dr + s[0]); hi[0] = std::max(hi[0], dr + s[0]);
    lo[1] = std::min(lo[1], dc + s[1]); hi[1] = std::max(hi[1], dc + s[1]);
  }
  if (lo[0] < -4 || hi[0] > 4 || lo[1] < -4 || hi[1] > 4 || row < C + hi[1] - lo[1]) return;
  g->in_place = true;
  g->self_row = (int)dr; g->self_col = (int)dc;
  g->halo[0] = (int)-lo[0]; g->halo[1] = (int)hi[0]; g->halo[2] = (int)-lo[1]; g->halo[3] = (int)hi[1];
  g->flat = 0; g->tail = 0; g->UC = 1; g->nt = 0; g->diag = 0;
  g->cphase = row % 4 == 0 ? (int)(((g->out_base % 4) + 4) % 4) : 0;
  g->xcd_remap = true;
  g->BX = std::min(64, std::max(4, next_pow2((C + g->cphase + 3) / 4)));
  g->BY = 256 / g->BX;
  const int64_t across = (C + g->cphase + 4 * g->BX - 1) / (4 * g->BX);
  g->VR = across * (R / (8 * (int64_t)g->BY)) >= 256 ? 8 : 4;
  if (saved_cells(*g).rows + saved_cells(*g).cols > (int64_t)1 << 30) g->in_place = false;
  g->in_place_once = g->in_place && c->opt_assign_in_place < 2 && in_place_tiles(*g) <= kOnceTiles;
}

// Products that are blocks of 32 x 32 from registers (gemm_block_body), before all other choices.
// - k over the waves of a workgroup: results of fewer than 16 tiles of 64 x 64, whatever the sum, and sums of up to 384 for up to 512 blocks, two
//   to a compute unit.  (us, tiles of 64 x 64 or 128 x 32 / this: 64^3 4.9 / 3.6, 300 x 46 x 320 5.3 / 3.4, with a bias and tanh 8.6 / 3.8, 46 x 296 x 320 10.6 /
//   4.9, 300^3 10.8 / 5.0, 500 x 300 x 500 10.9 / 5.2, 1000 x 350 x 500 11.2 / 8.8; 625 blocks of 800 x 300 x 800 11.2 / 10.6, 1024 of 1000 x 200 x 1000
//   9.3 / 11.1.  Longer sums: 256 x 512 x 256 9.9 / 6.3, but 512^3 11.3 / 9.5 to 13 by layout: from 16 tiles on all of them stay.)  Long sums are split over
//   workgroups as well: by 0.0062 us per value of k and round of 256 blocks (420 x 3250 x 124 transposed by 3, 4, 5, 9 parts: 168 workgroups 14.1, 224 12.4, 280 17.0, 504 13.7),
//   2.7 for the second launch and 0.08 per part that it adds up (97 x 1491 x 40 10.3 / 8.1,
//   50 x 4800 x 32 11.8 / 9.4, 200 x 500 x 200, unsplit, 10.8 / 6.0).  From about 2000 values of k per workgroup on tiles would be faster (320 x 8192 x 192 20.5 / 20,
//   320 x 16384 x 192 31.5 / 35, 192 x 49000 x 192 50 / 58) with larger errors (3.0e-7 / 2.2e-7, 4.1e-7 / 3.0e-7, 5.4e-7 / 3.8e-7: chains four times as long) and four
//   times the partial results: these sums stay here.
// - waves side by side: more blocks, ragged operands, sums of up to 32 and at most 10^7 results (100000 x 9 x 40 13.5 / 9.6, 30000 x 20 x 200 13.4 / 12, 3000 x 20 x 3000 16.1 / 13.9,
//   4936 x 27 x 1131 14.1 / 11.8; 2000 x 33 x 4000 15.8 / 16.7, 16384 x 16 x 4096 53 / 64), and sums of up to 128 whose results pass through a function of many
//   instructions, which the larger tiles run when their products are done (tanh: 4936 x 27 x 1131 27.5 / 17.3, 11845 x 48 x 2066 77 / 60, 16384 x 100 x 1000 82 / 61,
//   4096 x 128 x 4096 91 / 64, 8000 x 64 x 1000 29.6 / 26.1, 5000 x 128 x 300 12.9 / 12.9).  Operands of 32 columns and fewer are read once by taller tiles.
static bool choose_gemm_blocks(GroupPlan* g) {
  const int64_t M = g->M, N = g->N, K = g->K;
  const int64_t blocks = ((M + 31) / 32) * ((N + 31) / 32), tiles = ((M + 63) / 64) * ((N + 63) / 64);
  if (tiles < 16 || (blocks <= 512 && K <= 384)) {
    double cost = 0;
    int best = 1;
    for (int ks = 1; ks <= g->slabs; ++ks) {
      const double us = (double)gemm_split_extent(K, ks) * 0.0062 * (double)((blocks * ks + 255) / 256) + (ks > 1 ? 2.7 + 0.08 * ks + (double)ks * (double)M * (double)N * 1.8e-6 : 0.0);
      if (ks == 1 || us < cost * 0.97) { cost = us; best = ks; }
    }
    g->UC = 8;
    g->BX = g->BY = 32;
    g->slabs = best;
  } else {
    int heavy = 0;   // (a division, a root, an exponential are a third of the others)
    for (const Instr& in : g->prog) if (heavy_op(in)) heavy += in.kind == IKind::UNARY && (in.op == GR_TANH || in.op == GR_ERF) ? 3 : 1;
    if (tiles >= (int64_t)1 << 24) return false;   // (a launch has fewer than 2^32 lanes; wider tiles are fewer)
    if (M <= 32 || N <= 32 || !((K <= 32 && M * N <= 10000000 && g->VR != 2) || (heavy >= 3 && K <= 128))) return false;
    g->UC = 1;
    g->BX = g->BY = 64;
    g->slabs = 1;
  }
  g->VR = 4;
  g->NP = 1;
  return true;
}

// The extents of a direct-to-LDS product that are not whole steps of k or groups of four (kGemmRestK, kGemmShiftM, kGemmShiftN).
int gemm_ragged(const GroupPlan& g) {
  return (g.K % 16 ? kGemmRestK : 0) + (g.groups[g.mat_group].coef[1] != 1 && g.M % 4 ? kGemmShiftM : 0) + (g.groups[g.vec_group].coef[0] != 1 && g.N % 4 ? kGemmShiftN : 0);
}

// Small or ragged matrix products: tiles of 64 x 64 (128 x 32, 32 x 128) with clamped loads (gemm_tile_body), after the
// choice between the kernels with tiles of 128 and 256.
// The split of K: cheapest by rounds of 256 workgroups times steps of 32 values of k at 0.62 us, 5 for the launch and the first
// loads, and for a split 4 for the second launch and the partial tiles' traffic at 5 TB/s.
// It takes over from the register-staged kernel (us, before / now: 2001^3 275 / 156, 649 x 448 x 714 26 / 15, 1792 x 74 x 213
// 14.6 / 6.3, 11845 x 2066 x 48 78 / 48, 2066 x 11845 x 48 62 / 39, 64 x 4096 x 4096 49 / 29, 30 x 5000 x 3000 56 / 23),
// except for short sums with a large result, whose stores bound it and which the larger tile writes faster (11845 x 48 x 2066
// 42 against 57, 16384 x 100 x 1000 44 / 58, 2^20 x 16 x 8 26 / 55), tall operands with few columns (65536 x 512 x 10 28 / 31)
// and large products of two operands contiguous along k (4001^3 1082 / 1111; the other layouts 1201 / 1143 and
// 1318 / 1152); and from the direct 128 x 128 kernel where an estimate of its time is lower than that kernel's (by 5 % where that one has one group of waves).  Both
// estimates, in microseconds: rounds of 256 workgroups times steps (fitted to 446 products of 64 to 4096 values of k in four layouts;
// that of the direct kernel where it multiplies pieces to 36), the launch, and for a split the second launch and the partial tiles' traffic; without a
// split the epilogue, which runs when the products are done (a second launch hides it behind its traffic): 4096 x 784 x 512 with a bias and
// tanh 40.5 clamped, 38 direct in two parts.  (us, direct / this: 512^3 15.5 / 11.3, 1024 x 512 x 512 17.5 / 14.2, 224 x 192 x 1856 12.8 / 8.5,
// 528 x 208 x 2320 14.7 / 14.7, 448 x 768 x 1456 23.0 / 22.8; stay: 368 x 2160 x 1296 28.3 / 32.8, 1296 x 3264 x 208 26.8 / 35.2, 3056 x 448 x 896 27.7 / 31.8,
// 2048^3 119 / 151.  The choice missed the faster one of 45 products by 7 % at most, 4096 x 784 x 512 plain 36.3 / 38.9.)
// Ragged extents (gemm_ragged) go to the direct kernel where it is estimated 7 % faster: always its two groups of waves and pieces, up to
// any number of workgroups; 4 more for every round, which stores before the next one loads, and 2 for the rest of k; `former` splits of K on
// the other side, as many as before they fitted the direct kernel, so that no chain gets longer.  Sums of fewer than 256 values for large results stay where they were.
// (us, 64 x 64 clamped / direct, errors against 64 bits: 1967 x 1499 x 1767 transposed 115 / 84, 4.9e-7 / 1.7e-7; 4729 x 589 x 749 transposed 51 / 40, 3.1e-7 / 1.2e-7;
// 1109 x 6941 x 349 65 / 56; 1779 x 1191 x 1699 72 / 66; 4177 x 1071 x 1371 121 / 118; 2599 x 157 x 7349 76 / 82; 1289 x 905 x 6105 144 / 151; 5091 x 459 x 817 49 / 58;
// 529 x 849 x 337 12.1 / 17.8: the last four stay.)
// `wanted`: splits of K that the larger tiles would take if they may store any number of partial tiles.  It decides
// between the kernels, so that a request that must not allocate takes the kernel that the same request would take
// otherwise (and that is loaded by then); g->slabs, which stays within its scratch array, bounds the splits.
void choose_gemm_tiles(GroupPlan* g, int wanted, int former) {
  const int64_t M = g->M, N = g->N, K = g->K;
  auto fits = [&](const AccessGroup& x, int kdim, int64_t other) {
    if (x.coef[kdim] == 1) return K >= 4;
    return x.coef[1 - kdim] == 1 && other >= 4 && x.coef[kdim] > 0 && x.coef[kdim] < ((int64_t)1 << 32);
  };
  if (M < 1 || N < 1 || K > (int64_t)1 << 30 || !fits(g->groups[g->mat_group], 1, M) || !fits(g->groups[g->vec_group], 0, N)) return;
  if (choose_gemm_blocks(g)) return;
  if (g->VR == 2 && g->BX != 128) return;
  const int64_t tm = N <= 32 ? 128 : (M <= 32 ? 32 : 64), tn = N <= 32 ? 32 : (M <= 32 ? 128 : 64);
  const int64_t tiles = ((M + tm - 1) / tm) * ((N + tn - 1) / tn);
  if (tiles > (int64_t)1 << 24) return;
  const int ragged = g->VR == 2 ? gemm_ragged(*g) : 0;
  if (g->VR != 2 || (ragged && K < 256)) {
    const bool rows_of_k = g->groups[g->mat_group].coef[1] == 1 && g->groups[g->vec_group].coef[0] == 1;
    if ((K <= 128 && M * N >= (int64_t)1 << 22) ||                   // stores
        (tn == 32 && tiles >= 256) ||                                // one pass over a tall operand
        (rows_of_k && M * N >= (int64_t)1 << 23)) {                  // many large tiles, both operands contiguous along k
      if (ragged) { g->VR = 1; g->slabs = former; }
      return;
    }
  }
  // Every accumulator adds two chains: at least half as many splits as the larger tiles would take, so that no chain gets
  // longer, and no more than those, so that the partial tiles need no more memory (of a request that must not allocate).
  double cost = 0;
  auto cheapest = [&](int before) {
    int best_ks = 0;
    for (int ks = (before + 1) / 2; ks <= before; ++ks) {
      const int64_t kch = gemm_split_extent(K, ks);
      const double rounds = (double)((tiles * ks + 255) / 256);
      const double us = rounds * (double)((kch + 31) / 32) * 0.62 + 5.0 + (ks > 1 ? 4.0 + (double)ks * (double)M * (double)N * 8.0 / 5e6 : 0.0);
      if (best_ks == 0 || us < cost * 0.97) { cost = us; best_ks = ks; }
    }
    return best_ks;
  };
  const int before = ragged ? former : g->slabs, best_ks = cheapest(before);
  if (g->VR == 2) {
    const int ks = cheapest(ragged ? former : wanted);
    auto rounds = [](int64_t workgroups) { return (double)((workgroups + 255) / 256); };
    auto split = [&](double launch, double traffic, int n) { return n > 1 ? launch + traffic * (double)n * (double)M * (double)N * 8e-6 : 0.0; };
    const int64_t wgs = ((M + 127) / 128) * ((N + 127) / 128) * wanted;
    const bool pieces = wgs <= 256 || ragged;   // (two groups of waves per workgroup, see gemm_big_body)
    const double direct = rounds(wgs) * (double)((gemm_split_extent(K, wanted) + 15) / 16) * (pieces ? 0.75 : 0.86) + (ragged ? 2.5 + 4.0 * rounds(wgs) : 4.5) + split(3.4, 0.18, wanted);
    const double clamped = rounds(tiles * ks) * (double)((gemm_split_extent(K, ks) + 31) / 32) * 0.56 + 4.0 + split(2.7, 0.22, ks);
    double epilogue = 0.0;   // vector instructions per result, at 39 of a lane per picosecond
    for (const Instr& in : g->prog)
      if (in.kind == IKind::UNARY || in.kind == IKind::BINARY) epilogue += heavy_op(in) ? 40.0 : 1.0;
    epilogue *= (double)M * (double)N / 3.9e7;
    if ((clamped + (ks > 1 ? 0.0 : epilogue)) * (ragged ? 0.93 : pieces ? 1.0 : 1.05) > direct + (wanted > 1 ? 0.0 : epilogue)) return;
  }
  g->VR = 3;
  g->UC = 1;
  g->BY = (int)tm;
  g->BX = (int)tn;
  g->NP = 1 + (M < tm && M % 4 ? 1 : 0) + (N < tn && N % 4 ? 2 : 0);   // (compiled in: groups of four that do not lie aligned in LDS)
  g->slabs = best_ks;
}

// Row-resident reductions: per-element values that are computed in one phase and used in a later one, the most alive
// between any two phases; `early`: one of them is computed, not just loaded, in the first.
int rowred_live(const GroupPlan& g, bool* early = nullptr) {
  const int n = (int)g.prog.size(), nst = (int)g.phases.size() + 1;
  std::vector<int> made(n, -1), used(n, -1);
  for (int s = 0; s < nst; ++s) {
    std::vector<int> work{s + 1 < nst ? g.phases[s].value : (g.results.empty() ? -1 : g.results[0])};
    std::vector<char> seen(n, 0);
    while (!work.empty()) {
      const int i = work.back();
      work.pop_back();
      if (i < 0 || seen[i]) continue;
      seen[i] = 1;
      used[i] = s;
      if (made[i] >= 0) continue;
      made[i] = s;
      work.push_back(g.prog[i].a);
      work.push_back(g.prog[i].b);
    }
  }
  int most = 0;
  for (int s = 0; s + 1 < nst; ++s) {
    int live = 0;
    for (int i = 0; i < n; ++i)
      if (!g.prog[i].uniform && made[i] >= 0 && made[i] <= s && used[i] > s) {
        ++live;
        if (s == 0 && early && g.prog[i].kind != IKind::LOAD) *early = true;
      }
    most = std::max(most, live);
  }
  return most;
}

// Whether rows of more than 16384 elements, which take one workgroup of 1024 lanes each, are worth keeping in registers
// over cutting the program at its reductions: estimates of both in microseconds, fitted to measurements at 1 to 600 rows of 16400
// to 65536 elements.  A workgroup walks its row in 0.5 per 10^4 elements and array read, 0.4 for a result per element and
// what divisions, exp and the like take; the chip holds 256 of them at a time.  Cuts cost a launch for each reduction and for
// the map after it (and before it, of a value that is used again), and the passes over the arrays between them at 5.5 TB/s.
// (us, cuts / resident: softmax of 8 x 20000 16.5 / 7.1, 16 x 65536 17.9 / 17.5, 1245 x 26936 148 / 58, 512 x 65536 133 / 62; x - mean(x) of 16 x 32768
// 8.8 / 4.0; tanh(0.79 x) x over the sum of its squares 16 x 20000 11.7 / 7.8, 16 x 65536 14.9 / 22.9, 64 x 65536 26.4 / 25.4; sum(tanh(x)) / 2 of 16 x 16400
// 8.6 / 5.4, 64 x 65536 10.6 / 17.7, 256 x 49152 16.7 / 14.9; sum(x) / 2 of 16 x 65536 8.7 / 5.0, 600 x 65536 30.9 / 27.6.)
bool long_rows_pay(const GroupPlan& g) {
  const int64_t C = g.dims[g.rank - 1];
  int64_t rows = 1;
  for (int k = 0; k + 1 < g.rank; ++k) rows *= g.dims[k];
  const bool full = !g.out_per_row;
  int loads = 0;
  double per = full ? 0.4 : 0.0;
  for (const Instr& in : g.prog) {
    if (in.uniform) continue;
    if (in.kind == IKind::LOAD) { ++loads; per += 0.5; }
    else if (heavy_op(in)) {
      if (in.op == GR_TANH || in.op == GR_ERF) per += full ? 1.5 : 1.8;
      else if (in.op == GR_EXP || in.op == GR_LOG) per += full ? 0.7 : 1.1;
      else per += 0.75;
    }
  }
  const int reds = (int)g.phases.size();
  bool stored = false;   // a value that is computed for the first reduction is used again
  rowred_live(g, &stored);
  const double resident = 2.7 + (double)C * per * 1e-4 * std::max(1.0, (double)rows / 256);
  const int launches = 2 * reds + (stored ? 1 : 0), passes = loads - 1 + (full ? 2 * reds + 2 + (stored ? 1 : 0) : 3 * reds - 2);
  const double cuts = std::max(4.1 * launches, 3.4 * launches + (double)rows * (double)C * 4.0 * passes / 5.5e6);
  return resident <= cuts;
}

// Vector instructions per element of a row's value, about; 0 for a program with an operation that is a sequence of its own
// (division, square root, exp, ...).
int simple_issue(const GroupPlan& g, const std::vector<char>& in_value) {
  int n = g.phases[0].out_dtype == GR_I64 ? 2 : (g.phases[0].op == GR_SUM ? 1 : (g.phases[0].in_dtype == GR_F32 ? 3 : 2));
  for (size_t i = 0; i < g.prog.size(); ++i) {
    const Instr& in = g.prog[i];
    if (!in_value[i]) continue;
    if (in.kind == IKind::UNARY) {
      if (in.op == GR_NEG || in.op == GR_ABS) n += in.dtype == GR_F32 ? 0 : 1;   // (modifiers of the instruction that reads them)
      else if (in.op == GR_SQUARE) n += in.dtype == GR_F32 ? 1 : 2;
      else return 0;
    } else if (in.kind == IKind::BINARY) {
      if (in.op == GR_ADD || in.op == GR_SUB) n += 1;
      else if (in.op == GR_MUL) n += in.dtype == GR_F32 ? 1 : 2;
      else if (in.op == GR_MAXIMUM || in.op == GR_MINIMUM) n += in.dtype == GR_F32 ? 3 : 2;
      else return 0;
    } else if (in.kind != IKind::LOAD && in.kind != IKind::CONST) return 0;
  }
  return n;
}

// Rows of at most 64 elements over two kept dimensions, each element a function of operands that follow the first
// of them and operands that follow the second: a lane per row of the longer one (see gen_rowred_pairs).
// (Squared distances, general kernel against this one, us: 262144 points to 32 centres in 16 dimensions 44.6 / 15.0, vector issue
// alone 11; 811856 x 7 x 38 284 / 32; 178688 x 27 x 47 205 / 24; 65536 x 64 x 64 79 / 24; 100000 x 8 x 8 5.3 / 5.1.  The row length is
// compiled in: beyond 64 elements the lane groups read whole lines of both operands and stay.)
// Where it loses, general / this one, us:
// - anything but additions, products, minima and the like: issue bounds both kernels, and K x 4 copies of an exp or a
//   division leave one wave per SIMD or spill (65536 x 32 x 64: sum of exp 72 / 173, of sqrt 63 / 127, of a log(a / b) 98 /
//   203, of exp(a - b) tanh(a b) 136 / 936; 200000 x 8 x 8: a / b 8.3 / 9.2);
// - long rows of several operands: their registers (three 300 x 3000 x 64 29 / 42; two 65536 x 32 x 64 55 / 35), or the
//   scalar unit's (two 200000 x 8 x 64 35 / 37), or many instructions for each (seven, 20000 x 64 x 64 28 / 29, 20000 x 16 x 32 5.2 / 7.5);
// - few pairs, which leave compute units idle: the cheapest programs below 2^17 (5000 x 16 x 64 4.5 / 5.6; 10000 x 16 x 64
//   7.0 / 5.7), 2^16 where the general kernel's lanes do not divide the row evenly (2000 x 64 x 48 6.9 / 4.2), others below 2^18 and with rows over 24 elements below 2^20 (cheb 20000 x 16 x 32 5.7 / 6.9; 20000 x 64 x 32 16.7 / 12.1);
// - rows of four, which the general kernel reads with one load each, unless the program is short (seven instructions 20000 x 64 4.4 / 4.9);
// - short rows whose results a lane stores, or reads, apart: 64-bit results and operands of the epilogue that follow both
//   dimensions, where the lane's is the outer one (i32 sums 65536 x 32 of 4 6.9 / 12.6, of 8 10.3 / 13.0, of 12 25.0 / 13.1; a matrix
//   added to 20000 x 64 of 8 7.8 / 8.6, of 12 18.6 / 8.5).
void choose_pair_rows(GroupPlan* g) {
  if (!g->out_per_row || g->phases.size() != 1 || g->rank != 3 || g->results.empty()) return;
  const int64_t K = g->dims[2], pairs = g->dims[0] * g->dims[1];
  if (K < 2 || K > 64 || g->NP != 1 || std::min(g->dims[0], g->dims[1]) < 4 || std::max(g->dims[0], g->dims[1]) < 256) return;
  const int ld = g->dims[0] >= g->dims[1] ? 0 : 1;
  auto value = [&](int root) {
    std::vector<char> seen(g->prog.size(), 0);
    std::vector<int> work{root};
    while (!work.empty()) {
      const int i = work.back();
      work.pop_back();
      if (i < 0 || seen[i]) continue;
      seen[i] = 1;
      work.push_back(g->prog[i].a);
      work.push_back(g->prog[i].b);
    }
    return seen;
  };
  const std::vector<char> in_value = value(g->phases[0].value);
  int held[2] = {0, 0};   // operands whose rows a lane holds, and that come through the scalar unit
  bool follows[2] = {false, false};
  for (size_t i = 0; i < g->prog.size(); ++i) {
    const Instr& in = g->prog[i];
    if (!in_value[i]) continue;
    if (in.dtype == GR_I64 || in.kind == IKind::RED) return;
    if (in.kind != IKind::LOAD) continue;
    const AccessGroup& ag = g->groups[in.group];
    if (!ag.structural_zero[0] && !ag.structural_zero[1]) return;
    if (ag.structural_zero[2]) continue;
    for (int d = 0; d < 2; ++d) if (!ag.structural_zero[d]) follows[d] = true;
    ++held[ag.structural_zero[ld] ? 1 : 0];
  }
  if (!follows[0] || !follows[1]) return;
  const int issue = simple_issue(*g, in_value);
  if (issue == 0 || issue > (K <= 4 ? 4 : (K <= 24 ? 8 : 5)) || held[0] * K > 128 || held[1] * K > 64) return;
  const bool cheap = issue <= 3 && held[0] == 1 && held[1] == 1;
  const bool ragged = K > 16 && K != 4 * (int64_t)g->row_threads;   // (the general kernel guards every element of such rows)
  if (pairs < (int64_t)1 << (cheap ? (ragged ? 16 : 17) : (K <= 24 ? 18 : 20))) return;
  bool apart = g->out_dtype == GR_I64;
  const std::vector<char> in_result = value(g->results[0]);
  for (size_t i = 0; i < g->prog.size(); ++i)
    if (in_result[i] && !in_value[i] && g->prog[i].kind == IKind::LOAD && !g->groups[g->prog[i].group].structural_zero[0] && !g->groups[g->prog[i].group].structural_zero[1]) apart = true;
  if (apart && ld == 0 && K <= 8) return;
  g->pair_k = (int)K;
  g->pair_lane = ld;
}

// REDUCE mode 0: how many lanes of a workgroup lie across the outputs (the rest along the reduced range) and
// how many workgroups share one output's range (their partial results are combined by a second launch).
// Bound by HBM for long ranges, by load latency times the elements one lane takes in turn for short ones: with a
// lane per four outputs and chunks of 256 elements (128 where the outputs were no multiple of four, scalar loads)
// few lanes ran and each waited for its loads 64 times over.  Standardisation of columns (two such sums and a map),
// before and after: 768 x 444 77.9 -> 15.7 us, 192 x 6848 61 -> 15, 112160 x 90 77.7 -> 56.8, 100003 x 257 109 -> 99
// (first sum 26 us = 4 TB/s, second 20 us), 3977 x 7342 110 -> 111; column sums of 4096 x 512 19 -> 9.
void choose_column_split(GroupPlan* g) {
  g->slabs = g->red_tight = 1;
  g->red_wide = false;
  if (g->red_out == 0) return;   // nothing to launch
  const int64_t V = reduce_units(*g), LEN = std::max<int64_t>(1, g->red_len);
  auto even = [&](int64_t bx) { const int64_t nb = (V + bx - 1) / bx; return (V + nb - 1) / nb; };   // blocks of equal width
  // One launch where that leaves a lane at most 32 elements, or where the outputs alone fill the chip: blocks as
  // wide as still give 512 workgroups, 16 lanes (256 bytes) at least; 256 where a block lies within one row; 128 of rows that are no
  // whole 128-byte lines, whose blocks share a line with each neighbour.  Long programs need the wavefronts there: 256, and 512 for few elements.
  // (us, blocks chosen by 512 workgroups / by this: 64 x 2^18 15.6 / 13.5, 32 x 2^19 15.1 / 12.9, 256 x 2^18 51.2 / 43.1, 512 x 2^19
  // 212 / 166, 2048 x 65536 91.5 / 84.4, 512 x 64 x 1024 over the middle 27.4 / 24.4, 700 x 70001 42.7 / 36.5 in 137 blocks and 47 in 274, of exp 46 /
  // 42 in 274 and 55 in 137; 20 x 300001 of exp 7.6 / 8.2 in 293; 64 x 64 x 64 x 64 over the third 14.0 / 17.8, whose rows are short.)
  bool heavy = false;
  for (const Instr& in : g->prog) if (heavy_op(in)) heavy = true;
  const int64_t D = g->dims[g->red_kept_rank - 1], fill = D < 1024 || (heavy && LEN < 64 && D % 32) ? 512 : (D % 32 == 0 || heavy ? 256 : 128);
  int64_t bx = kReduceLanes;
  while (bx > 16 && (V + bx - 1) / bx < fill) bx /= 2;
  g->red_bx = (int)even(bx);
  const bool full = bx >= 64 && (V + bx - 1) / bx >= fill;
  g->red_wide = full && LEN > 8 * (kReduceLanes / g->red_bx);   // (fewer elements per lane: all of them at once)
  if (full || LEN <= 32 * (kReduceLanes / g->red_bx)) return;
  // Otherwise enough chunks for two workgroups per compute unit, of 16 elements per lane at least.  Rows of whole
  // 128-byte lines: blocks of 32 lanes (8192^2 47.5 us; 16 lanes 50.5, 64 52.3, 128 58.9, 256 62.9; 16384 x 4096 50.6, 52.4,
  // 58.3, 60.6, 73.1); ragged rows: whole rows up to 128 lanes, else 64 (100003 x 257 22.5 us with 65 lanes, 24.0 with 33,
  // 27.5 with 22; 3977 x 7342 30.1 with 32, 28.6 with 64, 29.4 with 128).  1024 or 2048 workgroups are no better.
  g->red_bx = (int)even(D % 32 == 0 ? 32 : (V <= 128 ? 128 : 64));
  const int64_t blocks = (V + g->red_bx - 1) / g->red_bx, by = kReduceLanes / g->red_bx;
  // (and never more than 256 elements in one lane's chain of additions)
  const int64_t nsplit = std::max<int64_t>(std::min<int64_t>((512 + blocks - 1) / blocks, std::max<int64_t>(1, LEN / (16 * by))), std::min<int64_t>((LEN + 256 * by - 1) / (256 * by), (int64_t)1 << 20));
  g->slabs = (int)nsplit;
  // Partial results of a request that must not allocate come out of the static scratch array, beside the request's
  // stored results.  Where they do not fit, it makes do with as many as chunks of 256 elements (128 where a lane owns one
  // output) by 256-lane workgroups would give.
  const bool quads = g->red_vec && D % 4 == 0;
  const int64_t few = ((quads ? g->red_out / 4 : g->red_out) + 255) / 256;
  g->red_tight = (int)std::min<int64_t>(nsplit, std::max<int64_t>(1, g->red_out < 64 && LEN >= 4096 ? std::min<int64_t>(2048 / g->red_out, LEN / 4096)
                                                                                                   : std::min<int64_t>(2048 / std::max<int64_t>(1, few), LEN / (quads ? 256 : 128))));
}

}  // namespace

// ---------------------------------------------------------------------------

// Operand of a contraction as an access group of its own.  The contraction kernels address it as
// base + i * coef[0] + j * coef[1]; the static shift that `load` keeps apart (a slice that starts
// at or beyond its step) is folded into the base here, and the group is never shared with another
// access: the other operand or an epilogue load may read the same array with the same map, but
// with coefficient slots that mean other dimensions or with another shift.
static int add_core_group(GroupPlan* g, const Builder& like, const Node* leaf, const IndexMap& lm) {
  GroupPlan tmp;
  std::vector<Instr> prog;
  Builder cb;
  cb.g = &tmp; cb.owned = like.owned; cb.rank = 2; cb.dims = like.dims; cb.prog = &prog;
  cb.load(leaf, lm);
  AccessGroup ag = tmp.groups[0];
  const Instr& ld = prog.back();
  for (int k = 0; k < 2; ++k) if (!ag.structural_zero[k]) ag.base += ag.coef[k] * ld.delta[k];
  ag.deltas.clear();
  ag.deltas.insert(std::vector<int64_t>(2, 0));
  g->groups.push_back(ag);
  return (int)g->groups.size() - 1;
}

static gr_status build_group(gr_ctx* c, Planner& pl, Node* r, GroupPlan* g, std::vector<Invalid>* invalid, bool force_generic = false) {
  NodeSet owned = pl.owned_by(r);
  g->root = r;
  g->out_dtype = r->dtype;
  g->nt = (int)c->opt_nontemporal;
  // An output of at least three quarters of the memory-side cache (256 MiB) is streamed out: its vector
  // stores carry the non-temporal hint as well (measured on MI355X: normalize 8192^2 93.9 ->
  // 86.7 us).  Smaller outputs stay cacheable for the sub-graph that reads them next (a 64 MiB
  // result that is consumed, or whose buffer is reused, within a few launches is 7-15 % slower
  // with hinted stores).
  // Only the value the request asked for: an intermediate result is read by the next sub-graph
  // of the same request at once.
  if (g->nt == 1 && r == pl.root && r->count() * (r->dtype == GR_I64 ? 8 : 4) >= (192ll << 20)) g->nt |= 8;

  // A root that already has data (the plain copy of an array into another buffer or through a
  // strided destination) is a map that loads it, whatever operation once produced it.
  if (r->materialized) owned.clear();

  // classify
  const Node* dot = nullptr;
  std::vector<const Node*> reds;
  for (const Node* n : owned) {
    if (n->kind == Kind::DOT && !small_dot(n)) { if (dot) { invalid->push_back({n, "second dot in one sub-graph"}); return GR_OK; } dot = n; }
    if (n->kind == Kind::REDUCE) reds.push_back(n);
  }
  if (dot && !reds.empty()) { invalid->push_back({dot, "dot mixed with a reduction"}); return GR_OK; }
  if (r->kind == Kind::RESHAPE && !r->materialized && (dot || !reds.empty())) {
    // a reshape is a row-major copy fused with pointwise producers only: reductions and contractions
    // below it are evaluated first and read as stored arrays
    if (dot) invalid->push_back({dot, "dot under a reshape"});
    for (const Node* n : reds) invalid->push_back({n, "reduction under a reshape"});
    return GR_OK;
  }

  Builder b;
  b.g = g;
  b.owned = &owned;

  if (r->kind == Kind::SCAN && !r->materialized) {
    // ---- map-scan: the operand expression is the map, the scan runs along one axis --------
    g->kind = GroupKind::SCAN;
    b.g->kind = GroupKind::SCAN;
    for (const Node* n : owned) if (n != r && (n->kind == Kind::REDUCE || (n->kind == Kind::DOT && !small_dot(n)) || n->kind == Kind::SCAN))
      invalid->push_back({n, "reduction, scan or dot under a scan"});
    if (!invalid->empty()) return GR_OK;
    const Node* x = r->in[0];
    int axis = 0;
    for (int d = 0; d < x->ndim; ++d) if (r->red_axis[d]) axis = d;
    // iteration space: the other dimensions in order, the scanned axis last
    int pos[MAXD], nk = 0;
    for (int d = 0; d < x->ndim; ++d) if (d != axis) { pos[d] = nk; g->orig_dims[nk++] = x->shape[d]; }
    pos[axis] = nk;
    g->orig_dims[nk] = x->shape[axis];
    const int n = nk + 1;
    g->orig_rank = n;
    b.rank = n; b.dims = g->orig_dims; b.prog = &g->prog;
    IndexMap xm(x->ndim);
    for (int d = 0; d < x->ndim; ++d) xm[d] = DimMap{pos[d], 1, 0};
    int v = b.eval(x, xm);
    if (!b.invalid.empty()) { *invalid = b.invalid; return GR_OK; }
    b.members_seen.insert(r);
    Phase p;
    p.op = r->op; p.in_dtype = x->dtype; p.out_dtype = r->dtype; p.value = v; p.node = r;
    g->phases.push_back(p);
    // the C-contiguous output takes part in dimension collapsing as one more access
    AccessGroup og;
    og.leaf = nullptr; og.dtype = r->dtype;
    for (int k = 0; k < MAXD; ++k) og.structural_zero[k] = true;
    { int64_t st = 1; for (int d = x->ndim - 1; d >= 0; --d) { og.coef[pos[d]] = st; og.structural_zero[pos[d]] = false; st *= x->shape[d]; } }
    og.deltas.insert(std::vector<int64_t>(n, 0));
    g->groups.push_back(og);
    std::vector<Instr>* ps[1] = {&g->prog};
    normalize_deltas(g, ps, 1, n);
    bool barrier[MAXD] = {false};
    if (nk > 0) barrier[nk - 1] = true;
    collapse_dims(g, barrier, ps, 1);
    if (g->orig_dims[n - 1] == 1 || g->collapse_to[n - 1] != g->rank - 1 || nk == 0) {
      // the scanned axis must remain the last collapsed dim even if its extent is 1
      if (g->orig_dims[n - 1] == 1) {
        bool only = true;
        for (int k = 0; k < nk; ++k) if (g->orig_dims[k] != 1) only = false;
        if (!only) { g->dims[g->rank] = 1; g->collapse_to[n - 1] = g->rank; g->rank++; }
      }
    }
    for (int k = 0; k < g->rank; ++k) g->out_coef[k] = g->groups.back().coef[k];
    g->groups.pop_back();
    const int sd = g->rank - 1;
    int64_t L = g->dims[sd], lines = 1;
    for (int k = 0; k < sd; ++k) lines *= g->dims[k];
    bool unit = g->out_coef[sd] == 1 || L == 1;
    for (const AccessGroup& ag : g->groups) if (!ag.structural_zero[sd] && ag.coef[sd] != 1) unit = false;
    g->scan_mode = unit ? 0 : 1;
    g->scan_nchunk = 1;
    g->scan_chunk = ((L + 1023) / 1024) * 1024;
    if (g->scan_mode == 0 && lines < 512 && L > 32768) {
      // long lines and few of them: reduce-then-scan over chunks (Section 3.2 refers to the
      // work-efficient scan: chunk sums, a scan of the sums, then the chunks with their offsets)
      int64_t want = std::max<int64_t>(1, 2048 / std::max<int64_t>(lines, 1));
      int64_t chunk = std::max<int64_t>(8192, (L + want - 1) / want);
      chunk = ((chunk + 1023) / 1024) * 1024;
      int64_t nch = (L + chunk - 1) / chunk;
      if (nch > 4096) { chunk = (((L + 4095) / 4096 + 1023) / 1024) * 1024; nch = (L + chunk - 1) / chunk; }
      g->scan_chunk = chunk;
      g->scan_nchunk = (int)nch;
      // 4-byte running values: one pass over the input with chained tiles of 8192 elements
      // (option "scan_one_pass" = 0 keeps the three kernels, which read the input twice)
      // tiles of 8192 elements, 20480 for lines of 2^25 elements and more (measured: 2^27 elements 200 us with 12288, 192-195 with 16384, 188 with 20480, 207 with 24576; option values from 2 to 24: 1024-element blocks per tile)
      const int64_t tile = 1024 * (c->opt_scan_one_pass >= 2 ? c->opt_scan_one_pass : (L >= ((int64_t)1 << 25) ? 20 : 8));
      if (c->opt_scan_one_pass && p.out_dtype != GR_I64 && tile <= 24576 && (L + tile - 1) / tile <= (int64_t)1 << 24) {
        g->scan_mode = 2;
        g->scan_chunk = tile;
        g->scan_nchunk = (int)((L + tile - 1) / tile);
      }
    }
    // four neighbouring lines per thread where the innermost line dimension is contiguous in every
    // array read and in the output, holds a multiple of four, and all values are 32 bits wide
    g->scan_vec = 0;
    if (g->scan_mode == 1 && sd >= 1 && g->dims[sd - 1] % 4 == 0 && g->out_coef[sd - 1] == 1 && p.in_dtype != GR_I64) {
      bool ok = true;
      for (const AccessGroup& ag : g->groups)
        if (ag.dtype == GR_I64 || (!ag.structural_zero[sd - 1] && ag.coef[sd - 1] != 1)) ok = false;
      for (const Instr& in : g->prog) if (in.dtype == GR_I64) ok = false;
      g->scan_vec = ok ? 1 : 0;
    }
    if (g->scan_vec) lines /= 4;   // threads per chunk
    // A thread walks its line eight steps at a time (eight loads in flight).  One pass over the
    // lines reads the input once and is kept down to scan_min threads (measured: 2^14 threads with
    // dwordx4 loads still beat the chunked form); below that the lines are cut into chunks so that
    // about scan_threads threads run.
    const int64_t scan_threads = c->opt_scan_threads > 0 ? c->opt_scan_threads : (g->scan_vec ? 65536 : 131072);
    const int64_t scan_min = c->opt_scan_min_threads > 0 ? c->opt_scan_min_threads : (g->scan_vec ? 16384 : 32768);
    int n_loads = 0;
    for (const Instr& in : g->prog) if (in.kind == IKind::LOAD) ++n_loads;
    if (g->scan_mode == 1 && g->scan_vec && lines > 0 && L >= 128 && c->opt_scan_one_pass && p.out_dtype != GR_I64 && n_loads <= 8) {
      // Lines of 128 positions or more, four of them per lane, 4-byte running values: ONE pass over
      // the input.  A workgroup keeps a tile of R positions along the scanned axis by W neighbouring
      // lines in registers (BX lanes across the lines, 256/BX lane groups along the axis, RPL
      // positions per lane), publishes the tile's totals and collects its offsets from the tiles
      // before it.  (Measured against a thread per four lines at every line count from 64 to 2^20:
      // the tiles win everywhere, by 5 % at 2^18 lines of 512 and by 2x at 2^16 lines of 1024.)
      const int64_t D = g->dims[sd - 1];
      int bx = 64;
      while (bx > 4 && (int64_t)bx * 4 > D) bx /= 2;   // W = 4*BX lines: at most D where D allows, at least 16
      const int ly = 256 / bx;
      const int64_t chains = (lines * 4 / D) * ((D + 4 * bx - 1) / (4 * bx));
      int rpl = n_loads <= 1 ? 32 : (n_loads <= 2 ? 16 : 8);
      while (rpl > 4 && chains * ((L + (int64_t)rpl * ly - 1) / ((int64_t)rpl * ly)) < 1024) rpl /= 2;
      const int64_t R = (int64_t)rpl * ly;
      const int64_t nch = (L + R - 1) / R;
      if (nch <= ((int64_t)1 << 20) && chains * nch <= ((int64_t)1 << 30)) {
        g->scan_mode = 3;
        g->BX = bx;
        g->scan_chunk = R;
        g->scan_nchunk = (int)nch;
        int grp = 4;
        while (grp < 64 && (int64_t)grp * grp < nch) grp *= 2;
        g->slabs = grp;   // tiles per group of the offset collection
      }
    }
    if (g->scan_mode == 1 && lines < scan_min && L >= 128) {
      // fewer lines than that: cut the lines into chunks (chunk totals, scan of the totals, chunks
      // with offsets, as above), which costs a second read of the input
      int64_t want = std::max<int64_t>(1, scan_threads / std::max<int64_t>(lines, 1));
      int64_t chunk = std::max<int64_t>(32, (L + want - 1) / want);
      int64_t nch = (L + chunk - 1) / chunk;
      if (nch > 4096) { chunk = (L + 4095) / 4096; nch = (L + chunk - 1) / chunk; }
      g->scan_chunk = chunk;
      g->scan_nchunk = (int)nch;
    }
    // Lines of up to 1024 elements: a lane group per line (16 lanes up to 256 elements, a wave beyond), see mode 4 of gen_scan.  A
    // workgroup per line leaves most of its lanes idle and pays a barrier and two LDS exchanges per line (2^25 values,
    // workgroup per line against lane groups, us: lines of 64 422 / 45, 144 200 / 47, 320 101 / 45, 703 69 / 49, 1024 47.6 / 45.0;
    // i32 to i64: lines of 100 329 / 80, 703 120 / 84).  Longer lines fill the workgroup (2048: 47 us).
    if (g->scan_mode == 0 && lines > 1 && L >= 4 && L <= 1024 && p.in_dtype != GR_I64 && n_loads <= 4) {
      bool narrow = true;
      for (const Instr& in : g->prog) if (in.dtype == GR_I64) narrow = false;
      if (narrow) {
        g->scan_mode = 4;
        g->BX = L <= 256 ? 16 : 64;
        g->NP = (int)((L + g->BX * 4 - 1) / (g->BX * 4));
        g->scan_chunk = 0;
      }
    }
    g->red_out = g->scan_vec ? lines * 4 : lines;
    g->red_len = L;
  } else if (dot && dot->ndim == 2) {
    // ---- matrix-matrix product on the matrix cores, with pointwise epilogue -----------------
    g->kind = GroupKind::GEMM;
    b.g->kind = GroupKind::GEMM;
    const Node* A = dot->in[0];
    const Node* B = dot->in[1];
    g->M = A->shape[0]; g->K = A->shape[1]; g->N = B->shape[1];
    if (r->ndim != 2 || r->shape[0] != g->M || r->shape[1] != g->N) { invalid->push_back({dot, "epilogue changes the shape"}); return GR_OK; }
    g->orig_rank = 2;
    g->orig_dims[0] = g->M; g->orig_dims[1] = g->N;
    b.rank = 2; b.dims = g->orig_dims; b.prog = &g->prog;
    IndexMap im(2);
    im[0] = DimMap{0, 1, 0}; im[1] = DimMap{1, 1, 0};
    int res = b.eval(r, im);
    if (!b.invalid.empty()) { *invalid = b.invalid; return GR_OK; }
    g->results.push_back(res);
    std::vector<Instr>* eps[1] = {&g->prog};
    normalize_deltas(g, eps, 1, 2);
    // operands: left in the space (m,k), right in the space (k,n); resolved through views only
    for (int side = 0; side < 2; ++side) {
      const Node* X = side == 0 ? A : B;
      int64_t cd[2] = {side == 0 ? g->M : g->K, side == 0 ? g->K : g->N};
      Builder cb;
      std::vector<Instr> scratch;
      cb.g = g; cb.owned = &owned; cb.rank = 2; cb.dims = cd; cb.prog = &scratch;
      IndexMap xm(2);
      xm[0] = DimMap{0, 1, 0}; xm[1] = DimMap{1, 1, 0};
      cb.canonicalize(X, xm);
      const Node* leaf; IndexMap lm;
      if (!resolve_to_leaf(X, xm, &leaf, &lm)) return fail(c, GR_ERR_UNSUPPORTED, "dot: operand is not materialised");
      // a private group per operand (an epilogue access or the other operand may read the same leaf
      // with the same map, but their coefficient slots mean different dimensions)
      (side == 0 ? g->mat_group : g->vec_group) = add_core_group(g, cb, leaf, lm);
      b.leaves_seen.insert(leaf);
    }
    b.members_seen.insert(dot);
    g->rank = 2;
    g->dims[0] = g->M; g->dims[1] = g->N;
    g->collapse_to[0] = 0; g->collapse_to[1] = 1;
    // few output tiles and a long contraction: split K over workgroups (about 512 of them, at
    // least 128 k per split); the partial tiles are combined by a second kernel
    g->slabs = 1;
    int former = 1;   // splits of K by what a product that does not fit the direct kernels takes
    int wanted = 0;   // splits of K by the direct 128 x 128 kernel if any number of partial tiles may be stored
    // columns of the output tile of one workgroup: 128, or 32 for narrow results and where the last
    // 128-wide tile would be more than half empty (measured, 65536 x 64 x 64: 14.5 us against 21.8 us;
    // 8192 x 512 x 520: 67 against 94 us; a full 128-wide tile costs about 0.3 of four 32-wide ones less)
    // (only where those empty columns are more than an eighth of the padded width: 4000 columns keep 128-wide tiles)
    {
      const int64_t padded = ((g->N + 127) / 128) * 128, pad = padded - g->N;
      g->BX = (g->N <= 96 || (pad >= 64 && pad * 8 > padded)) ? 32 : 128;
    }
    if (c->opt_gemm_bn == 32 || c->opt_gemm_bn == 128) g->BX = (int)c->opt_gemm_bn;
    // k extent of one step of the main loop (one barrier per step): 16, or 32 on request
    g->UC = (g->BX == 128 && c->opt_gemm_kstep == 32) ? 2 : 1;
    {
      const int64_t tiles = ((g->M + 127) / 128) * ((g->N + g->BX - 1) / g->BX);
      if (tiles > 0 && tiles < 192 && g->K >= 256) {
        int64_t ks = std::min<int64_t>(512 / tiles, g->K / 128);
        if (ks >= 2) g->slabs = (int)std::min<int64_t>(ks, 256);
      }
      if (c->opt_gemm_split >= 1) g->slabs = (int)std::min<int64_t>(std::min<int64_t>(c->opt_gemm_split, 256), std::max<int64_t>(1, g->K / 32));
    }
    // Large products of operands that are contiguous along one of their two dimensions: 256 x 256 tiles, one
    // workgroup per compute unit, tiles loaded straight into LDS (BX = 256 selects that kernel).  It needs
    // whole steps of 16 values of k, a result that fills most of its rounds over the 256 compute units, and lane offsets
    // of 32 bits: an operand contiguous along k is loaded in rows of its
    // other dimension (row stride below 2^21 elements), one contiguous along its other dimension in rows of k
    // (stride below 2^24).
    {
      const AccessGroup& ag = g->groups[g->mat_group];
      const AccessGroup& bg = g->groups[g->vec_group];
      const int64_t tiles = ((g->M + 255) / 256) * ((g->N + 255) / 256), rounds = (tiles + 255) / 256;
      // other: the extent of the operand's dimension that is not k (a multiple of four where that dimension is the
      // contiguous one: its elements are loaded in groups of four)
      auto fits = [](const AccessGroup& x, int kdim) {   // kdim: which of the operand's two dimensions is k
        if (x.structural_zero[0] || x.structural_zero[1]) return false;
        const int64_t sk = x.coef[kdim], so = x.coef[1 - kdim];
        if (sk == 1 && so != 1) return so >= 16 && so < ((int64_t)1 << 21);
        if (so == 1 && sk != 1) return sk >= 128 && sk < ((int64_t)1 << 24);
        return false;
      };
      // Edge tiles are whole tiles of work: the result must fill 85 % of its rounds over the 256 compute units, 65 %
      // where M or N is not a multiple of 128 (the 128-wide kernel's guarded edge tiles make it slower there; measured
      // on 4000^3: 136 against 97 TFLOP/s, 8000^3: 144 against 114, 10000 x 4096 x 10000, seven rounds 85 % full: 126 against 117).
      const int64_t need = (g->M % 128 == 0 && g->N % 128 == 0) ? 17 : 13;
      // (ragged extents, see below: two groups of waves, whose sums of pieces stay nearer 64 bits than the two float32 chains of clamped tiles; one of
      // the other kernels would not: 1470 x 832 x 1216 transposed 2.7e-7 clamped, 3.6e-7 with one float32 chain)
      const int ragged = gemm_ragged(*g);
      former = g->slabs;
      const bool direct = c->opt_gemm_big && c->opt_gemm_bn == 0 && g->K >= 32 && fits(ag, 1) && fits(bg, 0);
      // (with K split over workgroups every split has to hold whole steps of k and at least two of them: the last one is the shortest)
      const bool split_ok = g->slabs == 1 || g->K - (g->slabs - 1) * gemm_split_extent(g->K, g->slabs) >= 32;
      if (direct && !ragged && g->slabs == 1 && g->M >= 256 && g->N >= 256 && g->M * g->N * 20 >= rounds * 256 * 65536 * need) {
        g->BX = 256;
        g->VR = 2;   // (marks the kernels whose tiles go straight into LDS)
        g->UC = 1;
      } else if (direct && g->BX == 128 && g->M >= 128 && g->N >= 128 && c->opt_gemm_split == 0) {
        // The same kernel with 128 x 128 tiles and K divided over `slabs`
        // workgroups per tile where that fills the compute units more evenly or at all.  The count is the one with the
        // lowest cost in a model fitted to measurements (microseconds): rounds of 256 workgroups times the
        // steps of one workgroup at 0.85 per step (two groups of waves, pieces) or 0.95 (one group, float32), plus, for a
        // split product, 6 for the second launch and the traffic of the partial tiles at 5 TB/s.  A larger count has to beat a smaller one
        // by 3 %.  Every split holds at least 128 values of k, the last one at least two steps; the partial tiles stay below 1 GiB
        // (within the static scratch array for a request that must not allocate).
        // (measured, us: 784 x 4096 x 512 by 8 splits 38.8, 44.4 with float32 instructions by 9; 2080 x 2368 x 512 by 3 50, 57 by 7;
        // 512 x 4096 x 512 by 16 27.2, 29.8; 1536^3 in one 78, by 3 (float32 instructions) 76; 3072^3 by 3 444, in one 525, float32 instructions both)
        const int64_t tiles128 = ((g->M + 127) / 128) * ((g->N + 127) / 128);
        auto cheapest = [&](int64_t room, int least) {   // room: floats of partial tiles
          double best = 0;
          int best_ks = 0;
          for (int ks = least; ks <= 64; ++ks) {
            const int64_t kch = gemm_split_extent(g->K, ks);
            if (ks > 1 && ragged && former <= 2) break;   // (clamped tiles may need no partial tiles there: a request that must not allocate fits then as before)
            if (ks > 1 && (kch < 128 || g->K - (ks - 1) * kch < 32 || (int64_t)ks * g->M * g->N > room)) continue;
            const int64_t wgs = tiles128 * ks, rnd = (wgs + 255) / 256, steps = (kch + 15) / 16;
            const double cost = (double)rnd * (double)steps * (wgs <= 256 || ragged ? 0.85 : 0.95) + (ks > 1 ? 6.0 + (double)ks * (double)g->M * (double)g->N * 8.0 / 5e6 : 0.0);
            if (best_ks == 0 || cost < best * 0.97) { best = cost; best_ks = ks; }
          }
          return best_ks;
        };
        wanted = cheapest((int64_t)1 << 28, 1);
        // (a request that must not allocate splits as well where the same request otherwise does: the kernel has it compiled in)
        const int best_ks = c->plan_static ? cheapest((int64_t)(c->static_cap / sizeof(float)), wanted > 1 ? 2 : 1) : wanted;
        g->slabs = std::max(1, best_ks);
        g->VR = 2;
        g->UC = 1;
      } else if (direct && split_ok && g->BX == 128 && g->M >= 128 && g->N >= 128) {
        // (a number of workgroups per tile set by option "gemm_split")
        g->VR = 2;
        g->UC = 1;
      }
    }
    if (c->opt_gemm_bn == 0 && c->opt_gemm_kstep == 0 && c->opt_gemm_split == 0 && c->opt_gemm_big && c->opt_gemm_clamped) choose_gemm_tiles(g, wanted ? wanted : g->slabs, former);
    // The direct kernel with 128 x 128 tiles (UC: groups of four waves in a workgroup): two groups divide a tile's steps and multiply pieces
    // where compute units have one workgroup each, one group with float32 instructions where they hold several at a time, which overlap
    // each other's loads, epilogues and arithmetic.
    // (us, one group / two: 256 workgroups or fewer: 4096 x 512 x 784 41.8 / 34.7, 2048^3 132 / 119.5, 512 x 2848 x 2352 70 / 60, 2048 x 128 x 2048
    // 14.8 / 13.3; more: 12800 x 64 x 768 22.1 / 26.1, 6000 x 128 x 1500 32.2 / 35.1, 12800 x 256 x 768 53.1 / 54.7,
    // 5120 x 384 x 2560 97 / 97, 3000 x 512 x 2048 66 to 71 / 62.)
    if (g->VR == 2) g->NP = 1 + gemm_ragged(*g);
    if (g->VR == 2 && g->BX == 128) g->UC = ((g->M + 127) / 128) * ((g->N + 127) / 128) * (wanted ? wanted : g->slabs) <= 256 || g->NP > 1 ? 2 : 1;
  } else if (dot && !(dot == r && dot_as_reduce(dot) && c->opt_fusion)) {
    // ---- contraction with pointwise epilogue ------------------------------
    g->kind = GroupKind::GEMV;
    const Node* A = dot->in[0];
    const Node* v = dot->in[1];
    g->K = v->shape[0];
    g->M = A->ndim == 2 ? A->shape[0] : 1;
    if (r->ndim != dot->ndim || (dot->ndim == 1 && r->shape[0] != dot->shape[0])) { invalid->push_back({dot, "epilogue changes the shape"}); return GR_OK; }
    g->orig_rank = 1;
    g->orig_dims[0] = g->M;
    b.rank = 1;
    b.dims = g->orig_dims;
    b.prog = &g->prog;
    IndexMap im(r->ndim);
    for (int d = 0; d < r->ndim; ++d) im[d] = DimMap{d, 1, 0};
    int res = b.eval(r, im);
    if (!b.invalid.empty()) { *invalid = b.invalid; return GR_OK; }
    g->results.push_back(res);
    // core operands, in the 2-D space (m, k); resolved through views only
    int64_t core_dims[2] = {g->M, g->K};
    Builder cb;
    cb.g = g; cb.owned = &owned; cb.rank = 2; cb.dims = core_dims;
    std::vector<Instr> scratch;
    cb.prog = &scratch;
    const Node* leaf; IndexMap lm;
    IndexMap am(A->ndim);
    if (A->ndim == 2) { am[0] = DimMap{0, 1, 0}; am[1] = DimMap{1, 1, 0}; } else am[0] = DimMap{1, 1, 0};
    cb.canonicalize(A, am);
    if (!resolve_to_leaf(A, am, &leaf, &lm)) return fail(c, GR_ERR_UNSUPPORTED, "dot: matrix operand is not materialised");
    // the epilogue's groups use 1-D coefficients; core groups are appended with (m,k) coefficients
    g->mat_group = add_core_group(g, cb, leaf, lm);
    b.leaves_seen.insert(leaf);
    IndexMap vm(1);
    vm[0] = DimMap{1, 1, 0};
    cb.canonicalize(v, vm);
    if (!resolve_to_leaf(v, vm, &leaf, &lm)) return fail(c, GR_ERR_UNSUPPORTED, "dot: vector operand is not materialised");
    g->vec_group = add_core_group(g, cb, leaf, lm);
    b.leaves_seen.insert(leaf);
    b.members_seen.insert(dot);
    g->rank = 1;
    g->dims[0] = g->M;
    g->collapse_to[0] = 0;
    const AccessGroup& mg = g->groups[g->mat_group];
    if (mg.coef[1] == 1 || g->K == 1) g->gemv_mode = 0;
    else if (mg.coef[0] == 1) g->gemv_mode = 1;
    else g->gemv_mode = 0;  // strided both ways: row-dot with scalar loads
    if (g->gemv_mode == 0) {
      g->LPR = g->K >= 2048 ? 64 : 16;
      int64_t per = (g->K + (int64_t)g->LPR * 4 - 1) / ((int64_t)g->LPR * 4);
      g->KV = (int)std::min<int64_t>(std::max<int64_t>(per, 1), 8);
    } else {
      g->BX = std::min(256, std::max(16, next_pow2((g->M + 3) / 4)));  // lanes across the output index
      g->BY = 256 / g->BX;
      int64_t colblocks = std::max<int64_t>(1, (g->M + (int64_t)g->BX * 4 - 1) / ((int64_t)g->BX * 4));
      // about one workgroup per CU measured best on MI355X (256 slabs: 78 us for 512 MiB, 1024: 85 us),
      // and fewer partial vectors make the second stage cheaper
      int64_t rows_per_slab = std::max<int64_t>((int64_t)g->BY * 8, (g->K + 255) / 256);
      int64_t slabs = std::max<int64_t>(1, (g->K + rows_per_slab - 1) / rows_per_slab);
      slabs = std::min<int64_t>(slabs, std::max<int64_t>(1, 256 / colblocks));
      if (c->opt_gemv_slabs > 0) slabs = std::min<int64_t>(c->opt_gemv_slabs, std::max<int64_t>(1, g->K));
      g->slabs = (int)slabs;
      g->unroll = c->opt_gemv_unroll == 16 ? 16 : (c->opt_gemv_unroll == 4 ? 4 : 8);
    }
    std::vector<Instr>* ps[1] = {&g->prog};
    // epilogue groups only: core groups carry no deltas
    normalize_deltas(g, ps, 1, 1);
  } else if (!reds.empty() || dot) {
    // Decide between row-resident and generic reduction.
    bool generic = dot != nullptr || force_generic;   // (a contraction planned as a reduction, see dot_as_reduce)
    if (r->kind == Kind::REDUCE) {
      const Node* x = r->in[0];
      bool last_only = x->ndim >= 1;
      for (int d = 0; d < x->ndim; ++d) if (r->red_axis[d] != (d == x->ndim - 1)) last_only = false;
      if (!last_only || x->shape[x->ndim - 1] > std::min<int64_t>(c->opt_rowred_max_cols, 16384)) generic = true;
    }
    if (generic) {
      // ---- generic reduction root: kept dims first, reduced dims last -----
      g->kind = GroupKind::REDUCE;
      for (const Node* n : reds) if (n != r) { invalid->push_back({n, "nested reduction under a generic reduction"}); }
      if (!invalid->empty()) return GR_OK;
      const Node* x = r->in[0];
      int pos[MAXD];
      int nk = 0;
      int v = -1;
      if (dot) {
        // iteration space (m, k) or (k): value A[m,k] * v[k], summed over k
        const Node* A = dot->in[0];
        const Node* vec = dot->in[1];
        if (A->ndim == 2) g->orig_dims[nk++] = A->shape[0];
        g->red_kept_rank = nk;
        g->orig_dims[nk] = vec->shape[0];
        g->orig_rank = nk + 1;
        b.rank = g->orig_rank; b.dims = g->orig_dims; b.prog = &g->prog;
        b.g->kind = GroupKind::REDUCE;
        int ids[2];
        for (int side = 0; side < 2; ++side) {
          const Node* X = side == 0 ? A : vec;
          IndexMap xm(X->ndim);
          if (X->ndim == 2) { xm[0] = DimMap{0, 1, 0}; xm[1] = DimMap{1, 1, 0}; } else xm[0] = DimMap{nk, 1, 0};
          b.canonicalize(X, xm);
          const Node* leaf; IndexMap lm;
          if (!resolve_to_leaf(X, xm, &leaf, &lm)) return fail(c, GR_ERR_UNSUPPORTED, "dot: operand is not materialised");
          ids[side] = b.load(leaf, lm);
        }
        Instr mul;
        mul.kind = IKind::BINARY; mul.op = GR_MUL; mul.dtype = GR_F32; mul.a = ids[0]; mul.b = ids[1];
        v = b.value_number(mul);
      } else {
      for (int d = 0; d < x->ndim; ++d) if (!r->red_axis[d]) { pos[d] = nk; g->orig_dims[nk++] = x->shape[d]; }
      g->red_kept_rank = nk;
      int nr = nk;
      for (int d = 0; d < x->ndim; ++d) if (r->red_axis[d]) { pos[d] = nr; g->orig_dims[nr++] = x->shape[d]; }
      g->orig_rank = nr;
      if (nr == 0) { g->orig_rank = 1; g->orig_dims[0] = 1; }
      b.rank = g->orig_rank; b.dims = g->orig_dims; b.prog = &g->prog;
      IndexMap xm(x->ndim);
      for (int d = 0; d < x->ndim; ++d) xm[d] = DimMap{pos[d], 1, 0};
      b.g->kind = GroupKind::REDUCE;
      v = b.eval(x, xm);
      }
      if (!b.invalid.empty()) { *invalid = b.invalid; return GR_OK; }
      b.members_seen.insert(r);
      Phase p;
      p.op = dot ? (int)GR_SUM : r->op; p.in_dtype = x->dtype; p.out_dtype = r->dtype; p.value = v; p.node = r;
      g->phases.push_back(p);
      std::vector<Instr>* ps[1] = {&g->prog};
      normalize_deltas(g, ps, 1, g->orig_rank);
      bool barrier[MAXD] = {false};
      if (nk > 0 && nk < g->orig_rank) barrier[nk - 1] = true;
      // kept/reduced boundary must survive extent-1 drops: recompute kept rank after collapsing
      collapse_dims(g, barrier, ps, 1);
      int kept_rank = 0;
      for (int k = 0; k < nk; ++k) if (g->collapse_to[k] >= 0) kept_rank = std::max(kept_rank, g->collapse_to[k] + 1);
      g->red_kept_rank = kept_rank;
      g->red_out = 1; g->red_len = 1;
      for (int k = 0; k < g->rank; ++k) (k < kept_rank ? g->red_out : g->red_len) *= g->dims[k];
      if (nk == g->orig_rank || (kept_rank == g->rank)) {
        // nothing left to reduce after dropping extent-1 dims: treat the single point as the reduced range
        g->red_len = 1;
      }
      // mode 0 (a thread per output) when consecutive outputs are consecutive in memory, mode 1
      // (a workgroup per output, lanes along the reduced range) when the reduced range is
      bool kept_unit = false, red_unit = false;
      for (const AccessGroup& ag : g->groups) {
        if (kept_rank > 0 && ag.coef[kept_rank - 1] == 1) kept_unit = true;
        if (g->rank > kept_rank && ag.coef[g->rank - 1] == 1) red_unit = true;
      }
      g->red_mode = (kept_unit && !red_unit) ? 0 : ((red_unit && !kept_unit) ? 1 : (g->red_out >= 4096 ? 0 : 1));
      // a handful of outputs whose elements are not contiguous: lanes across them would leave most of a workgroup's
      // loads apart, so the lanes go along the reduced range even though it is strided
      if (g->red_mode == 0 && !kept_unit && g->red_out < 64 && g->red_len >= 4096) g->red_mode = 1;
      // mode 0 with four consecutive outputs per lane: the innermost kept dimension is contiguous
      // (or absent) in every array read, has four elements or more, and all values are 32 bits wide
      g->red_vec = 0;
      if (g->red_mode == 0 && kept_rank >= 1 && g->dims[kept_rank - 1] >= 4 && p.in_dtype != GR_I64) {
        bool ok = true;
        for (const AccessGroup& ag : g->groups)
          if (ag.dtype == GR_I64 || (!ag.structural_zero[kept_rank - 1] && ag.coef[kept_rank - 1] != 1)) ok = false;
        for (const Instr& in : g->prog) if (in.dtype == GR_I64) ok = false;
        g->red_vec = ok ? 1 : 0;
      }
      // mode 1 over several reduced dimensions: four consecutive elements per lane as long as they
      // cannot straddle the innermost one
      if (g->red_mode == 1 && g->rank > kept_rank + 1 && g->dims[g->rank - 1] % 4 == 0) g->red_vec = 1;
      // split the reduced range so that about 2048 workgroups run (two-stage reduction, Section 3.2)
      if (g->red_mode == 0) choose_column_split(g);
      else {
        const int64_t nsplit = std::min<int64_t>(std::max<int64_t>(1, 2048 / std::max<int64_t>(g->red_out, 1)), std::max<int64_t>(1, g->red_len / 4096));
        g->slabs = (int)std::min<int64_t>(nsplit, 4096);
      }
    } else {
      // ---- row-resident reductions fused with producers and consumers -----
      g->kind = GroupKind::ROWRED;
      // the reduction recorded last (nearest to the root, possibly the root itself) fixes the row
      // space; reductions over any other space become sub-graphs of their own
      const Node* x = reds.back()->in[0];
      for (const Node* n : reds) {
        const Node* xo = n->in[0];
        bool same = xo->ndim == x->ndim;
        for (int d = 0; same && d < x->ndim; ++d) if (xo->shape[d] != x->shape[d]) same = false;
        if (!same) invalid->push_back({n, "reductions over different row spaces"});
      }
      if (!invalid->empty()) return GR_OK;
      int n = x->ndim;
      g->orig_rank = n;
      for (int d = 0; d < n; ++d) g->orig_dims[d] = x->shape[d];
      // root shape must be the row space, or one value per row
      bool full = r->ndim == n, per_row_keep = r->ndim == n, per_row_drop = r->ndim == n - 1;
      for (int d = 0; d < n; ++d) {
        if (full && r->shape[d] != x->shape[d]) full = false;
        if (per_row_keep && r->shape[d] != (d == n - 1 ? 1 : x->shape[d])) per_row_keep = false;
        if (per_row_drop && d < n - 1 && r->shape[d] != x->shape[d]) per_row_drop = false;
      }
      if (x->shape[n - 1] == 1) per_row_keep = false;  // degenerate: full covers it
      if (!full && !per_row_keep && !per_row_drop) {
        for (const Node* q : reds) invalid->push_back({q, "consumer shape differs from the row space"});
        return GR_OK;
      }
      g->out_per_row = !full;
      b.rank = n; b.dims = g->orig_dims; b.prog = &g->prog;
      IndexMap im(r->ndim);
      for (int d = 0; d < r->ndim; ++d) im[d] = DimMap{d, 1, 0};
      int res = b.eval(r, im);
      if (!b.invalid.empty()) { *invalid = b.invalid; return GR_OK; }
      g->results.push_back(res);
      std::vector<Instr>* ps[1] = {&g->prog};
      normalize_deltas(g, ps, 1, n);
      bool barrier[MAXD] = {false};
      if (n >= 2) barrier[n - 2] = true;  // never merge rows into the reduced axis
      collapse_dims(g, barrier, ps, 1);
      // the reduced axis must remain the last collapsed dim even if its extent is 1
      if (g->orig_dims[n - 1] == 1) {
        g->dims[g->rank] = 1;
        g->collapse_to[n - 1] = g->rank;
        g->rank++;
        if (g->rank == 2 && g->dims[0] == 1 && g->collapse_to[0] < 0 && n == 1) {}
      }
      int64_t C = g->dims[g->rank - 1];
      // few vec4 positions per lane keep the register count low and the occupancy high
      // (measured on MI355X for 4096-float rows: 256 lanes 93 us, 128 lanes 96 us, 64 lanes 104 us)
      // lanes per row: enough for one to four dwordx4 positions per lane; very short rows share a
      // wave between many rows instead of leaving most of 16 lanes idle
      // Rows of more than 16384 elements: 1024 lanes, up to 16 positions per lane, one workgroup per row, where that pays
      // (long_rows_pay).  A sum of such rows that is a result of its own stays with the two-stage kernel.
      g->row_threads = C <= 4 ? 1 : (C <= 8 ? 2 : (C <= 16 ? 4 : (C <= 32 ? 8 : (C <= 256 ? 16 : (C <= 1024 ? 64 : (C <= 2048 ? 128 : 256))))));
      if (c->opt_rowred_threads == 16 || c->opt_rowred_threads == 64 || c->opt_rowred_threads == 128 || c->opt_rowred_threads == 256)
        if (C <= c->opt_rowred_threads * 64) g->row_threads = (int)c->opt_rowred_threads;  // at most 16 positions per lane
      if (C > 16384) g->row_threads = 1024;
      g->NP = (int)std::max<int64_t>(1, (C + (int64_t)g->row_threads * 4 - 1) / ((int64_t)g->row_threads * 4));
      // The values that a phase leaves for later ones live in registers: of 128 per lane, 80 may hold them (the others hold
      // the operands and temporaries of a few positions).
      if (g->row_threads == 1024 && ((int64_t)rowred_live(*g) * g->NP * 4 > 80 || !long_rows_pay(*g))) {
        for (const Node* n : reds) if (n != r) invalid->push_back({n, "rows too long to keep their values"});
        if (!invalid->empty()) return GR_OK;
      }
      // Rows that run along a strided axis of every array read while another axis is the contiguous
      // one (an array stored transposed): lanes along such a row would each touch another cache
      // line.  The reductions are evaluated by the generic kernel instead, which gives a thread
      // to each output and walks the lanes along the contiguous axis.
      if (g->row_threads > 1) {
        const int cd = g->rank - 1;
        bool inner_unit = false, outer_unit = false;
        for (const AccessGroup& ag : g->groups) {
          if (!ag.structural_zero[cd] && ag.coef[cd] == 1) inner_unit = true;
          for (int k = 0; k < cd; ++k) if (!ag.structural_zero[k] && ag.coef[k] == 1 && g->dims[k] > 1) outer_unit = true;
        }
        if (!inner_unit && outer_unit) {
          if (reds.size() == 1 && reds[0] == r) {
            *g = GroupPlan();
            return build_group(c, pl, r, g, invalid, true);
          }
          for (const Node* n : reds) if (n != r) invalid->push_back({n, "reduction along a strided axis"});
          if (!invalid->empty()) return GR_OK;
        }
      }
      // Short rows (up to 64 elements) reduced to one value each: a wave that owns only 4 to 64 rows lives about as long as
      // its loads take, and the waves a SIMD can hold then bound the rate.  Each lane group takes four
      // rows, the loads of all four in flight together, the four results stored at the end.
      int64_t rows = 1;
      for (int k = 0; k + 1 < g->rank; ++k) rows *= g->dims[k];
      g->row_iters = (g->out_per_row && C <= 64 && rows >= (int64_t)1 << 18 && c->opt_rowred_rows != 1) ? 4 : 1;  // (measured: 2 and 8 rows are no better, 256-element rows lose)
      if (c->opt_rowred_threads == 0 && c->opt_rowred_rows == 0) choose_pair_rows(g);
      if (c->opt_rowred_rows > 1 && g->out_per_row && g->row_threads <= 64) g->row_iters = (int)std::min<int64_t>(c->opt_rowred_rows, 8);
    }
  } else {
    // ---- map ----------------------------------------------------------------
    g->kind = GroupKind::MAP;
    for (const Node* n : reds) invalid->push_back({n, "reduction inside a map sub-graph"});
    if (!invalid->empty()) return GR_OK;
    // A reshape root is the row-major copy of its operand: the sub-graph iterates over the operand's
    // index space and writes a C-contiguous buffer, which is the result under either shape.
    const Node* src = map_source(r);
    int n = std::max(src->ndim, 1);
    g->orig_rank = n;
    if (src->ndim == 0) g->orig_dims[0] = 1;
    for (int d = 0; d < src->ndim; ++d) g->orig_dims[d] = src->shape[d];
    IndexMap im(src->ndim);
    for (int d = 0; d < src->ndim; ++d) im[d] = DimMap{d, 1, 0};
    // Single-point program: enough to learn the accesses, fix the schedule and key the
    // kernel cache.  The per-lane patch program is a function of exactly these and is only
    // built when the cache misses (expand_patch).
    b.rank = n; b.dims = g->orig_dims; b.prog = &g->prog1;
    g->result1 = b.eval(src, im);
    if (src != r) b.members_seen.insert(r);
    if (!b.invalid.empty()) { *invalid = b.invalid; return GR_OK; }
    // where the elements go: a C-contiguous buffer, or the strided destination of a slice assignment
    // (whose strides are given in the root's own shape: not for a reshape root)
    if (r == pl.root && pl.out && r->ndim > 0 && src == r) {
      g->out_base = pl.out->base;
      for (int d = 0; d < r->ndim; ++d) g->out_orig_coef[d] = pl.out->strides[d];
    } else {
      int64_t st = 1;
      for (int d = n - 1; d >= 0; --d) { g->out_orig_coef[d] = st; st *= g->orig_dims[d]; }
    }
    push_output_group(g, n);
    std::vector<Instr>* ps[1] = {&g->prog1};
    normalize_deltas(g, ps, 1, n);
    bool barrier[MAXD] = {false};
    collapse_dims(g, barrier, ps, 1);
    pop_output_group(g);
    choose_map_schedule(c, g, !(r == pl.root && pl.out));
    if (r == pl.root && pl.out && pl.out->in_place && src == r && r->ndim > 0) choose_in_place(c, g);
    g->owned.assign(owned.begin(), owned.end());
  }

  for (const Node* n : b.members_seen) g->members.push_back(n);
  std::sort(g->members.begin(), g->members.end(), [](const Node* a, const Node* b2) { return a->id < b2->id; });
  for (const Node* n : b.leaves_seen) g->leaves.push_back(n);
  std::sort(g->leaves.begin(), g->leaves.end(), [](const Node* a, const Node* b2) { return a->id < b2->id; });
  if (g->pair_k) {
    const int k = g->pair_k, ld = g->pair_lane;
    g->pair_k = g->pair_lane = 0;
    make_signature(g);
    g->general = g->signature;
    g->pair_k = k;
    g->pair_lane = ld;
  }
  make_signature(g);
  return GR_OK;
}

// Builds the patch program of a MAP sub-graph: the point function evaluated at every
// point of the per-lane patch (VR rows x UC chunks of 4 columns), with values shared
// between points (broadcast operands, overlapping slice views) computed once.
gr_status expand_patch(gr_ctx* c, GroupPlan* g) {
  if (g->kind != GroupKind::MAP || !g->prog.empty()) return GR_OK;
  Node* r = g->root;
  const int n = g->orig_rank;
  // innermost original dims of the last two collapsed dims carry the patch shifts
  int col_dim = -1, row_dim = -1;
  for (int k = 0; k < n; ++k) {
    if (g->collapse_to[k] == g->rank - 1) col_dim = k;
    if (g->rank >= 2 && g->collapse_to[k] == g->rank - 2) row_dim = k;
  }
  if (col_dim < 0) col_dim = n - 1;
  GroupPlan tmp;
  tmp.kind = GroupKind::MAP;
  tmp.root = r;
  tmp.orig_rank = n;
  for (int k = 0; k < n; ++k) tmp.orig_dims[k] = g->orig_dims[k];
  tmp.consts = g->consts;
  Builder b;
  const NodeSet owned(g->owned.begin(), g->owned.end());
  b.g = &tmp; b.owned = &owned; b.rank = n; b.dims = tmp.orig_dims; b.prog = &tmp.prog;
  const Node* src = map_source(r);
  IndexMap im(src->ndim);
  for (int d = 0; d < src->ndim; ++d) im[d] = DimMap{d, 1, 0};
  const bool was_planned = r->planned;  // the root is computed here, not read
  r->planned = false;
  for (int v = 0; v < g->VR; ++v)
    for (int u = 0; u < g->UC; ++u)
      for (int j = 0; j < 4; ++j) {
        IndexMap pm = im;
        for (int d = 0; d < src->ndim; ++d) {
          if (d == col_dim) pm[d].off += (int64_t)u * g->BX * 4 + j;
          if (d == row_dim) pm[d].off += v;
        }
        // shifted points are evaluated as if the root were larger; the root's own extent-1
        // dims stay canonicalised to index 0, which is right: such dims carry no shift
        tmp.results.push_back(b.eval(src, pm));
      }
  r->planned = was_planned;
  if (!b.invalid.empty()) return fail(c, GR_ERR_UNSUPPORTED, "map: patch expansion met an unexpected node");
  tmp.out_dtype = g->out_dtype;
  for (int k = 0; k < n; ++k) tmp.out_orig_coef[k] = g->out_orig_coef[k];
  push_output_group(&tmp, n);
  std::vector<Instr>* ps[1] = {&tmp.prog};
  normalize_deltas(&tmp, ps, 1, n);
  bool barrier[MAXD] = {false};
  // the patch shifts touch only dims that are innermost in their runs, so the collapse
  // decision of the single-point program is reproduced
  collapse_dims(&tmp, barrier, ps, 1);
  pop_output_group(&tmp);
  bool same = tmp.rank == g->rank && tmp.groups.size() == g->groups.size() && tmp.consts.size() == g->consts.size();
  for (size_t i = 0; same && i < tmp.groups.size(); ++i)
    if (tmp.groups[i].ident != g->groups[i].ident || tmp.groups[i].base != g->groups[i].base) same = false;
  if (!same) {
    std::ostringstream m;
    m << "map: patch expansion disagrees with the single-point program (rank " << tmp.rank << "/" << g->rank << ", groups "
      << tmp.groups.size() << "/" << g->groups.size() << ", consts " << tmp.consts.size() << "/" << g->consts.size() << ")";
    return fail(c, GR_ERR_UNSUPPORTED, m.str());
  }
  g->prog.swap(tmp.prog);
  g->results.swap(tmp.results);
  return GR_OK;
}

// A row-dot contraction z = A.v whose (epilogue) result r is the vector operand of the
// column-accumulate contraction A^T.r over the same matrix needs the matrix only once: the
// two sub-graphs become one kernel pass (the row stays in registers between the two
// contractions).  This goes one step further than the paper, which runs every contraction
// as its own library call; the sub-graph list, the materialised nodes and the values are
// the same.
static void fuse_gemv_pairs(gr_ctx* c, Plan* plan) {
  if (!c->opt_gemv_pair || !c->opt_fusion) return;
  for (size_t i = 0; i + 1 < plan->groups.size(); ++i) {
    GroupPlan& A = *plan->groups[i];
    GroupPlan& B = *plan->groups[i + 1];
    if (A.kind != GroupKind::GEMV || B.kind != GroupKind::GEMV || A.gemv_mode != 0 || B.gemv_mode != 1) continue;
    const AccessGroup& ma = A.groups[A.mat_group];
    const AccessGroup& mb = B.groups[B.mat_group];
    const AccessGroup& vb = B.groups[B.vec_group];
    bool same_matrix = ma.leaf == mb.leaf && ma.base == mb.base && ma.coef[1] == 1 && mb.coef[0] == 1 && ma.coef[0] == mb.coef[1] &&
                       A.M == B.K && A.K == B.M;
    bool feeds = vb.leaf == A.root && vb.base == 0 && vb.coef[1] == 1;
    if (!same_matrix || !feeds || A.K > 2048 || A.M < 1) continue;
    // Lanes of a row, and rows that they take at a time.  32 columns and fewer leave half of 16 lanes without any (us, 16 / 8 lanes: 1000000 x 16 31.1 /
    // 22.9, 300001 x 27 14.9 / 13.2).  Six rows where a lane holds four columns (two, four, six, eight rows: 378142 x 41 24.0, 18.0, 15.7, 17.2; 1000000 x 16 27.8,
    // 20.4, 17.7, 20.0), two beyond (one, two, four: 524288 x 128 62.9, 43.7, 45.7; 100000 x 200 24.9, 18.5, 20.1; 20000 x 1500 28.9, 25.9, 29.2); one where whole 16-byte
    // loads of wide rows fill a long range, which reads at HBM's rate so (262144 x 512 86.0 / 87.3, 131072 x 1024 81.6 / 84; 60000 x 448 24.9 / 22.7, 20000 x 2048 34.1 / 32.6)
    // and for rows of three columns, without 16 bytes.
    A.LPR = A.K <= 32 ? 8 : A.K <= 512 ? 16 : 64;
    A.KV = (int)std::max<int64_t>(1, (A.K + (int64_t)A.LPR * 4 - 1) / ((int64_t)A.LPR * 4));
    const bool whole = A.KV >= 4 && A.K % (A.LPR * 4) == 0 && A.M > 16 * 512 * (256 / A.LPR);
    A.unroll = A.K < 4 || whole ? 1 : (A.KV == 1 ? 6 : 2);
    int rpb = 256 / A.LPR;
    int64_t slabs = std::min<int64_t>(512, (A.M + rpb - 1) / rpb);  // measured: 256 -> 115 us, 512 -> 94 us, 1024 -> 96 us, 4096 -> 109 us
    if (c->opt_gemv_slabs > 0) slabs = std::min<int64_t>(c->opt_gemv_slabs, (A.M + rpb - 1) / rpb);
    A.slabs = (int)std::max<int64_t>(1, slabs);
    B.slabs = A.slabs;
    A.gemv_mode = 2;
    A.pair = std::move(plan->groups[i + 1]);
    plan->groups.erase(plan->groups.begin() + i + 1);
    make_signature(&A);
  }
}

// Do instruction `a` of A's program and `b` of B's compute the same value?  `known`: pairs compared before (values used more than
// once are reached over many paths, twice as many per level of a chain of squares).
static bool same_value(const GroupPlan& A, int a, const GroupPlan& B, int b, std::map<std::pair<int, int>, bool>* known) {
  if (a < 0 || b < 0) return a == b;
  const auto at = known->find({a, b});
  if (at != known->end()) return at->second;
  const Instr& x = A.prog[a];
  const Instr& y = B.prog[b];
  bool same = x.kind == y.kind && x.op == y.op && x.dtype == y.dtype;
  if (same && x.kind == IKind::LOAD) {
    const AccessGroup& p = A.groups[x.group];
    const AccessGroup& q = B.groups[y.group];
    int64_t off = p.base - q.base;
    same = p.leaf == q.leaf;
    for (int k = 0; same && k < A.rank; ++k) {
      same = p.coef[k] == q.coef[k];
      off += p.coef[k] * (x.delta[k] - y.delta[k]);
    }
    same = same && off == 0;
  } else if (same && x.kind == IKind::CONST) {
    same = std::memcmp(&A.consts[x.cslot].value, &B.consts[y.cslot].value, sizeof(double)) == 0;
  } else if (same) {
    same = same_value(A, x.a, B, y.a, known) && same_value(A, x.b, B, y.b, known);
  }
  (*known)[{a, b}] = same;
  return same;
}

// Column sums S of v whose mean is what the next sub-graph takes v's squared deviations from (var, std and what divides by
// them): sums of (v - S / n)^2 with n the reduced elements.  One pass over the operands gives both; the sub-graph list, the
// materialised nodes and the sums are the same.  Bound by HBM like the sums alone; a launch or two less for small arrays.
// (us for a variance, two passes / one: 100003 x 257 44.4 / 28.6, 8192^2 93.6 / 51.5, 3977 x 7342 55 / 36, 16384 x 512 18.3 / 14.1, 3000 x 1000 18.6 / 14.1,
// 768 x 444 14.8 / 10.3, 64 x 8192 9.9 / 8.5, 1000003 x 4 20.3 / 17.1, 100 x 30 8.8 / 8.7; column standardisation of 100003 x 257 88 / 73.)
// Where the sums take the wide kernel (outputs enough to fill the chip in one launch each) they stay apart, and where the partial results,
// three per split instead of one for each sum, could crowd the static scratch array: where they are large, and where the request
// fits it with the sums apart and not with them together.  So do those of many arrays, whose values the registers of 512 lanes do not hold beside
// the means and squares (us, two passes / one, 20011 x 514 by arrays: of exp 12 241 / 192, 16 311 / 303, 20 382 / 403, 24 485 / 580; of
// sums 16 293 / 162, 32 623 / 453, 40 888 / 792).
static void fuse_moments(gr_ctx* c, Plan* plan, const Node* root) {
  if (!c->opt_moments || !c->opt_fusion) return;
  for (size_t i = 0; i + 1 < plan->groups.size(); ++i) {
    GroupPlan& A = *plan->groups[i];
    GroupPlan& B = *plan->groups[i + 1];
    if (A.kind != GroupKind::REDUCE || B.kind != GroupKind::REDUCE || A.pair || B.pair || A.red_mode != 0 || B.red_mode != 0 || A.red_wide || A.red_vec != B.red_vec) continue;
    if (A.rank != B.rank || A.red_kept_rank != B.red_kept_rank || A.red_len < 2 || A.red_len >= (int64_t)1 << 24 || A.red_out < 1 || A.red_out != B.red_out) continue;
    bool same = true;
    for (int k = 0; k < A.rank; ++k) same = same && A.dims[k] == B.dims[k];
    if (!same || (A.slabs > 1 && (int64_t)A.red_tight * A.red_out * 12 > (int64_t)4 << 20)) continue;
    const Phase& pa = A.phases[0];
    const Phase& pb = B.phases[0];
    if (pa.op != GR_SUM || pb.op != GR_SUM || pa.out_dtype != GR_F32 || pb.out_dtype != GR_F32 || pa.in_dtype != GR_F32 || pb.in_dtype != GR_F32) continue;
    int loads = 0;
    bool heavy = false;
    for (const Instr& in : A.prog) {
      loads += in.kind == IKind::LOAD;
      heavy = heavy || heavy_op(in);
    }
    if (loads > (heavy ? 16 : 40)) continue;
    const Instr& q = B.prog[pb.value];
    int d = -1;
    if (q.kind == IKind::UNARY && q.op == GR_SQUARE) d = q.a;
    else if (q.kind == IKind::BINARY && q.op == GR_MUL && q.a == q.b) d = q.a;
    if (d < 0 || B.prog[d].kind != IKind::BINARY || B.prog[d].op != GR_SUB) continue;
    const Instr& m = B.prog[B.prog[d].b];
    if (m.kind != IKind::BINARY || m.op != GR_DIV || B.prog[m.b].kind != IKind::CONST || B.consts[B.prog[m.b].cslot].value != (double)A.red_len) continue;
    const Instr& s = B.prog[m.a];
    if (s.kind != IKind::LOAD || B.groups[s.group].leaf != A.root) continue;
    // S is read at the output's own position
    const AccessGroup& sg = B.groups[s.group];
    int64_t at = sg.base, st = 1;
    bool own = true;
    for (int k = A.rank - 1; k >= 0; --k) {
      at += sg.coef[k] * s.delta[k];
      if (k >= A.red_kept_rank) { own = own && (sg.coef[k] == 0 || A.dims[k] == 1); continue; }
      own = own && (sg.coef[k] == st || A.dims[k] == 1);
      st *= A.dims[k];
    }
    std::map<std::pair<int, int>, bool> known;
    if (!own || at != 0 || !same_value(A, pa.value, B, B.prog[d].a, &known)) continue;
    const size_t apart[2] = {scratch_need(*plan, root, false), scratch_need(*plan, root, true)};
    A.pair = std::move(plan->groups[i + 1]);
    plan->groups.erase(plan->groups.begin() + i + 1);
    bool crowded = false;
    for (int tight = 0; tight < 2; ++tight) crowded = crowded || (apart[tight] <= kStaticScratchBytes && scratch_need(*plan, root, tight != 0) > kStaticScratchBytes);
    if (crowded) plan->groups.insert(plan->groups.begin() + i + 1, std::move(A.pair));   // (A stays where it is: the list has had this length)
    else make_signature(&A);
  }
}

gr_status make_plan_uncached(gr_ctx* c, Node* root, Plan* plan) {
  if (root->kind == Kind::SCALAR) return fail(c, GR_ERR_UNSUPPORTED, "a bare scalar cannot be materialised");
  Planner pl;
  pl.c = c;
  pl.root = root;
  pl.out = plan->out;
  pl.collect();
  pl.initial_cuts();
  for (int iter = 0; iter < 10000; ++iter) {
    if (!pl.assign_owners()) continue;
    clear_planned(plan);
    plan->groups.clear();
    std::vector<Invalid> invalid;
    bool restart = false;
    std::vector<Node*> order;
    for (Node* n : pl.sub) if (pl.cuts.count(n)) order.push_back(n);
    if (!pl.cuts.count(root) || root->materialized) order.push_back(root);  // root with data: a plain copy
    std::sort(order.begin(), order.end(), [](Node* a, Node* b) { return a->id < b->id; });
    order.erase(std::unique(order.begin(), order.end()), order.end());
    for (Node* r : order) {
      std::unique_ptr<GroupPlan> g(new GroupPlan());
      gr_status st = build_group(c, pl, r, g.get(), &invalid);
      if (st != GR_OK) { clear_planned(plan); plan->groups.clear(); return st; }
      if (!invalid.empty()) {
        bool added = false;
        for (const Invalid& iv : invalid) if (pl.cuts.insert(iv.node).second) added = true;
        if (!added) { clear_planned(plan); plan->groups.clear(); return fail(c, GR_ERR_UNSUPPORTED, "cannot plan: " + invalid[0].why); }
        restart = true;
        break;
      }
      plan->groups.push_back(std::move(g));
      if (!r->materialized) {
        // later sub-graphs read this node as a C-contiguous leaf
        r->planned = true;
        int64_t s = 1;
        for (int d = r->ndim - 1; d >= 0; --d) { r->strides[d] = s; s *= r->shape[d]; }
        r->offset = 0;
        plan->planned_nodes.push_back(r);
      }
    }
    if (!restart) {
      plan->out_honoured = !plan->out || (!plan->groups.empty() && plan->groups.back()->root == root && plan->groups.back()->kind == GroupKind::MAP &&
                                          map_source(root) == root);
      fuse_gemv_pairs(c, plan);
      fuse_moments(c, plan, root);
      return GR_OK;
    }
  }
  clear_planned(plan);
  plan->groups.clear();
  return fail(c, GR_ERR_UNSUPPORTED, "planner did not converge");
}

void clear_planned(Plan* plan) {
  for (Node* n : plan->planned_nodes) n->planned = false;
  plan->planned_nodes.clear();
}

std::string describe_plan(const Plan& plan) {
  std::ostringstream s;
  int i = 0;
  for (const auto& gp : plan.groups) {
    const GroupPlan& g = *gp;
    const char* kn = g.kind == GroupKind::MAP ? "MAP" : g.kind == GroupKind::ROWRED ? "ROWRED" : g.kind == GroupKind::REDUCE ? "REDUCE" : g.kind == GroupKind::SCAN ? "SCAN" : g.kind == GroupKind::GEMM ? "GEMM" : "GEMV";
    s << '#' << i++ << ' ' << kn << " root=" << g.root->id << " shape=(";
    for (int d = 0; d < g.root->ndim; ++d) s << (d ? "," : "") << g.root->shape[d];
    s << ") iter=(";
    for (int d = 0; d < g.rank; ++d) s << (d ? "," : "") << g.dims[d];
    s << ") members=[";
    bool first = true;
    for (const Node* n : g.members) {
      if (n->is_view()) continue;
      s << (first ? "" : ",") << n->id << ':' << node_label(n);
      first = false;
    }
    s << "] leaves=[";
    first = true;
    for (const Node* n : g.leaves) { s << (first ? "" : ",") << n->id; first = false; }
    s << "] loads=" << [&] { int k = 0; for (const Instr& in : (g.kind == GroupKind::MAP ? g.prog1 : g.prog)) if (in.kind == IKind::LOAD) ++k; return k; }();
    if (g.kind == GroupKind::GEMM) s << " M=" << g.M << " N=" << g.N << " K=" << g.K << " tile=" << (g.VR >= 3 ? g.BY : g.BX == 256 ? 256 : 128) << "x" << g.BX << (g.VR == 4 ? (g.UC > 1 ? " clamped, k over waves" : " clamped, from registers") : g.VR == 3 ? " clamped" : g.VR == 2 ? " direct" : "");
    if (g.kind == GroupKind::GEMM && g.slabs > 1) s << " split=" << g.slabs;
    if (g.kind == GroupKind::GEMV) s << " mode=" << (g.gemv_mode == 2 ? "row-dot+column-accumulate" : (g.gemv_mode ? "column-accumulate" : "row-dot")) << " M=" << g.M << " K=" << g.K;
    if (g.pair) {
      s << " fused-with=[root=" << g.pair->root->id << " members=[";
      bool f2 = true;
      for (const Node* n : g.pair->members) { if (n->is_view()) continue; s << (f2 ? "" : ",") << n->id << ':' << node_label(n); f2 = false; }
      s << "]]";
    }
    if (g.kind == GroupKind::REDUCE) {
      if (g.red_mode == 0) s << " lanes=" << g.red_bx << "x" << kReduceLanes / g.red_bx << (g.red_vec ? " by four outputs" : "") << (g.red_wide ? " wide" : "");
      else s << " workgroup per output";
      if (g.slabs > 1) s << " splits=" << g.slabs;
    }
    if (g.kind == GroupKind::ROWRED) {
      s << " phases=" << g.phases.size() << " row_threads=" << g.row_threads << " NP=" << g.NP;
      if (g.pair_k) s << " pairs: length=" << g.pair_k << " lanes_along=" << g.pair_lane;
      else if (g.row_iters > 1) s << " rows_per_group=" << g.row_iters;
    }
    if (g.kind == GroupKind::SCAN) s << " mode=" << (g.scan_mode == 4 ? "lines-in-lane-groups" : g.scan_mode == 3 ? "one-pass-line-tiles" : (g.scan_mode == 2 ? "one-pass-tiles" : (g.scan_mode ? "thread-per-line" : "lanes-along-axis"))) << " lines=" << g.red_out << " length=" << g.red_len << " chunks=" << g.scan_nchunk;
    if (g.kind == GroupKind::MAP && g.flat == 1) s << " lanes over groups of columns patch=" << g.VR << "x4";
    else if (g.kind == GroupKind::MAP) s << " tile=" << g.BY * g.VR << "x" << g.BX * 4 * g.UC << " patch=" << g.VR << "x" << g.UC * 4 << (g.flat == 2 ? " overlapping" : "") << (g.in_place ? " in place" : "");
    s << '\n';
  }
  return s.str();
}

int square_root_of(const GroupPlan& g, int s) {
  const Phase& ph = g.phases[s];
  if (g.kind != GroupKind::ROWRED || g.row_threads == 1024 || ph.op != GR_SUM || ph.in_dtype != GR_F32 || ph.out_dtype != GR_F32 || ph.value < 0) return -1;
  const Instr& v = g.prog[ph.value];
  if (!(v.kind == IKind::UNARY && v.op == GR_SQUARE) && !(v.kind == IKind::BINARY && v.op == GR_MUL && v.a == v.b)) return -1;
  // (a square that an earlier phase has computed is kept, its root may not be)
  std::vector<char> seen(g.prog.size(), 0);
  std::vector<int> work;
  for (int q = 0; q < s; ++q) work.push_back(g.phases[q].value);
  while (!work.empty()) {
    const int i = work.back();
    work.pop_back();
    if (i < 0 || seen[i]) continue;
    seen[i] = 1;
    work.push_back(g.prog[i].a);
    work.push_back(g.prog[i].b);
  }
  return seen[ph.value] ? -1 : v.a;
}

}  // namespace gr
