// Kernel generator: turns one planned sub-graph into HIP source for gfx950.
//
// Section 3 of the paper generates, from a point function and an iteration
// space, a `map` kernel (one GPU thread per point) or a `map-reduce` kernel
// (per-block combine in shared memory, second kernel for the block partials).
// The skeletons below keep that contract (the point function is the SSA
// program built by the planner) and replace the launch shapes with ones
// fitted to CDNA4:
//
//   MAP     each lane owns a patch of VR rows x UC chunks of 4 consecutive
//           columns; loads and stores are dwordx4; values shared between the
//           points of a patch (broadcast operands, overlapping slice views)
//           are loaded and computed once per patch and stay in registers.
//   ROWRED  a row is held in registers by 16 / 64 / 256 lanes across all
//           reduction phases and the final map (wave shuffles, LDS only
//           across the four waves of a 256-lane row).
//   REDUCE  generic reduction root: a thread or a workgroup per output.
//   GEMV    bandwidth-bound contraction kernels (row-dot, and
//           column-accumulate with a deterministic second combine stage in
//           the manner of the paper's two-kernel reduction) whose epilogue
//           is the point function of the dot's pointwise consumers.
#include "codegen.h"

#include <algorithm>
#include <functional>
#include <map>
#include <set>
#include <sstream>

#include "ctx.h"

namespace gr {

char access_class(const AccessGroup& ag, int dim) {
  if (ag.structural_zero[dim]) return 'Z';
  if (ag.coef[dim] == 1 && ag.dtype != GR_I64) return '1';
  return 'G';
}

// Arrays that are streamed through once (unit stride, not re-read through shifted
// views, not broadcast along rows) bypass cache retention; operands that lanes
// share stay cacheable.
bool nontemporal_group(const GroupPlan& g, int group) {
  const AccessGroup& ag = g.groups[group];
  if ((g.nt & 7) == 0 || ag.dtype == GR_I64) return false;
  if (g.kind == GroupKind::GEMV) return group == g.mat_group;
  if (g.kind == GroupKind::GEMM) return false;  // operand tiles are re-read by other workgroups: keep them cacheable
  // (tiles of neighbouring lines of a scan: lanes run along the innermost line dimension)
  const int lane_dim = g.kind == GroupKind::SCAN && g.scan_mode == 3 ? g.rank - 2 : g.rank - 1;
  if (access_class(ag, lane_dim) != '1') return false;
  if ((g.nt & 7) >= 2) return true;
  if (ag.deltas.size() > 1) return false;
  // read once = the operand follows every outer iteration dimension; one that is broadcast along
  // any of them is read again by other rows or planes and stays cacheable
  for (int k = 0; k < g.rank; ++k) if (k != lane_dim && ag.structural_zero[k]) return false;
  return true;
}

ArgLayout arg_layout(const GroupPlan& g) {
  ArgLayout L;
  int s = 0;
  for (size_t i = 0; i < g.groups.size(); ++i) {
    bool core = (g.kind == GroupKind::GEMV || g.kind == GroupKind::GEMM) && ((int)i == g.mat_group || (int)i == g.vec_group);
    int nc = core ? 2 : g.rank;
    L.ptr.push_back(s++);
    L.base.push_back(s++);
    L.coef.push_back(s);
    L.ncoef.push_back(nc);
    s += nc;
  }
  L.out = s++;
  L.dims = s;
  s += g.rank;
  L.consts = s;
  s += (int)g.consts.size();
  L.extra = s;
  s += 4;
  L.ocoef = s;
  if (g.kind == GroupKind::SCAN || g.kind == GroupKind::MAP) s += g.rank;
  if (g.kind == GroupKind::GEMM) s += 2;  // split-K: workspace pointer, k extent of one split
  L.obase = s;
  if (g.kind == GroupKind::MAP) s += 1;
  L.total = s;
  return L;
}

std::string kernel_name(const GroupPlan& g) {
  switch (g.kind) {
    case GroupKind::MAP: return g.in_place_once ? "gr_map_save_store" : "gr_map";
    case GroupKind::ROWRED: return "gr_rowred";
    case GroupKind::REDUCE: return "gr_reduce";
    case GroupKind::SCAN: return "gr_scan";
    case GroupKind::GEMM: return "gr_gemm";
    case GroupKind::GEMV: return g.gemv_mode == 2 ? "gr_gemv_pair" : (g.gemv_mode ? "gr_gemv_colacc" : "gr_gemv_rowdot");
  }
  return "gr_kernel";
}

namespace {

const char* cty(gr_dtype dt) { return dt == GR_F32 ? "float" : (dt == GR_I32 ? "int" : "long long"); }
const char* vty4(gr_dtype dt) { return dt == GR_F32 ? "f4u" : "i4u"; }
const char* vty2(gr_dtype dt) { return dt == GR_F32 ? "f2u" : "i2u"; }

struct Em {
  const GroupPlan& g;
  ArgLayout L;
  std::ostringstream o;
  int slot_base = 0;     // first slot of this sub-graph's block inside the kernel's argument array
  int total_slots = 0;   // size of the whole argument array
  std::string qp = "q";  // name prefix of the per-group base pointers
  explicit Em(const GroupPlan& gp) : g(gp), L(arg_layout(gp)) { total_slots = L.total; }
  std::string slot(int n) const { return "a.s[" + std::to_string(slot_base + n) + "]"; }

  // *(const T*)(addr), with the non-temporal hint where the group streams
  std::string ld(int group, const std::string& type, const std::string& addr) const {
    if (nontemporal_group(g, group)) return "__builtin_nontemporal_load((const GM " + type + "*)(" + addr + "))";
    return "*(const GM " + type + "*)(" + addr + ")";
  }

  std::string S(int n) const { return "((long long)" + slot(n) + ")"; }
  std::string dim(int k) const { return S(L.dims + k); }
  std::string cst(int cslot) const {
    const ConstSlot& c = g.consts[cslot];
    std::string s = slot(L.consts + cslot);
    if (c.dtype == GR_F32) return "__uint_as_float((unsigned)" + s + ")";
    if (c.dtype == GR_I32) return "((int)" + s + ")";
    return "((long long)" + s + ")";
  }
  std::string coef(int grp, int k) const { return S(L.coef[grp] + k); }

  static std::string unop(int op, gr_dtype dt, const std::string& x) {
    if (dt == GR_F32) switch (op) {
      case GR_NEG: return "(-" + x + ")";
      case GR_ABS: return "__builtin_fabsf(" + x + ")";
      case GR_EXP: return "gr_expf(" + x + ")";
      case GR_LOG: return "gr_logf(" + x + ")";
      case GR_SQRT: return "gr_sqrtf(" + x + ")";
      case GR_SQUARE: return "(" + x + " * " + x + ")";
      case GR_TANH: return "gr_tanhf(" + x + ")";
      case GR_ERF: return "gr_erff(" + x + ")";
    }
    switch (op) {  // i32: two's-complement wrap-around through unsigned arithmetic
      case GR_NEG: return "((int)(0u - (unsigned)" + x + "))";
      case GR_ABS: return "(" + x + " < 0 ? (int)(0u - (unsigned)" + x + ") : " + x + ")";
      case GR_SQUARE: return "((int)((unsigned)" + x + " * (unsigned)" + x + "))";
    }
    return "0";
  }
  static std::string binop(int op, gr_dtype dt, const std::string& x, const std::string& y) {
    if (dt == GR_F32) switch (op) {
      case GR_ADD: return "(" + x + " + " + y + ")";
      case GR_SUB: return "(" + x + " - " + y + ")";
      case GR_MUL: return "(" + x + " * " + y + ")";
      case GR_DIV: return "(" + x + " / " + y + ")";
      case GR_MAXIMUM: return "gr_maxf(" + x + ", " + y + ")";
      case GR_MINIMUM: return "gr_minf(" + x + ", " + y + ")";
    }
    switch (op) {
      case GR_ADD: return "((int)((unsigned)" + x + " + (unsigned)" + y + "))";
      case GR_SUB: return "((int)((unsigned)" + x + " - (unsigned)" + y + "))";
      case GR_MUL: return "((int)((unsigned)" + x + " * (unsigned)" + y + "))";
      case GR_MAXIMUM: return "(" + x + " >= " + y + " ? " + x + " : " + y + ")";
      case GR_MINIMUM: return "(" + x + " <= " + y + " ? " + x + " : " + y + ")";
    }
    return "0";
  }

  // combine(acc, x) for a reduction phase
  static std::string combine(const Phase& p, const std::string& acc, const std::string& x) {
    if (p.op == GR_SUM) {
      if (p.out_dtype == GR_I64) return "(" + acc + " + (long long)" + x + ")";
      return "(" + acc + " + " + x + ")";
    }
    if (p.in_dtype == GR_F32) return std::string(p.op == GR_MAX ? "gr_maxf(" : "gr_minf(") + acc + ", " + x + ")";
    return "(" + acc + (p.op == GR_MAX ? " >= " : " <= ") + x + " ? " + acc + " : " + x + ")";
  }
  // acc combined with the value of phase `s`, whose name (or, of a sum of squares, its root's) `name` gives
  template <class F>
  static std::string accumulate(const GroupPlan& g, int s, const std::string& acc, const F& name) {
    const Phase& p = g.phases[s];
    const int root = square_root_of(g, s);
    if (root >= 0) return "__builtin_fmaf(" + name(root) + ", " + name(root) + ", " + acc + ")";
    return combine(p, acc, name(p.value));
  }
  static std::string identity(const Phase& p) {
    if (p.op == GR_SUM) return p.out_dtype == GR_F32 ? "0.0f" : (p.out_dtype == GR_I64 ? "0ll" : "0");
    if (p.in_dtype == GR_F32) return p.op == GR_MAX ? "(-__builtin_inff())" : "__builtin_inff()";
    return p.op == GR_MAX ? "(-2147483647 - 1)" : "2147483647";
  }
  static std::string zero(gr_dtype dt) { return dt == GR_F32 ? "0.0f" : (dt == GR_I64 ? "0ll" : "0"); }
};

// gr_erff, gr_divc: the text the interpreter kernels are compiled from as well
#define GR_DEVICE_MATH_SOURCE(...) #__VA_ARGS__
const char* const kDeviceMath =
#include "device_math.h"
    ;
const char* const kDeviceTanh =
#include "device_tanh.h"
    ;
#undef GR_DEVICE_MATH_SOURCE

bool calls(const GroupPlan& g, int op) {
  for (const std::vector<Instr>* p : {&g.prog, &g.prog1})
    for (const Instr& in : *p) if (in.kind == IKind::UNARY && in.op == op) return true;
  return false;
}

void prelude(Em& e) {
  // every pointer the kernels dereference is a global-memory pointer (arguments arrive as
  // integers, so the address space has to be stated for global_load/global_store to be used)
  e.o << "#define GM __attribute__((address_space(1)))\n"
         "typedef float f4 __attribute__((ext_vector_type(4)));\n"
         "typedef f4 f4u __attribute__((aligned(4)));\n"
         "typedef float f2 __attribute__((ext_vector_type(2)));\n"
         "typedef f2 f2u __attribute__((aligned(4)));\n"
         "typedef int i4 __attribute__((ext_vector_type(4)));\n"
         "typedef i4 i4u __attribute__((aligned(4)));\n"
         "typedef int i2 __attribute__((ext_vector_type(2)));\n"
         "typedef i2 i2u __attribute__((aligned(4)));\n"
         "struct Args { unsigned long long s[" << e.total_slots << "]; };\n"
         // linear index -> coordinates: rem % d with rem /= d, in 32-bit arithmetic whenever both fit
         // (a 64-bit division is a long instruction sequence, paid per row or per element)
         "static __device__ __forceinline__ long long gr_peel(long long& rem, long long d) {\n"
         "  if ((((unsigned long long)rem) | ((unsigned long long)d)) >> 32) { const long long i = rem % d; rem /= d; return i; }\n"
         "  const unsigned r = (unsigned)rem, dd = (unsigned)d, q = r / dd;\n  rem = q;\n  return r - q * dd;\n}\n"
         // the math helpers' test for a rare argument somewhere in the wave and the barrier that keeps its
         // block a branch; straight-line code in matrix-product kernels, whose epilogues run over up to
         // 256 accumulators per lane and would spill around branches, and in the matrix-vector kernels, whose
         // epilogue sits in the loop over rows: a wave-wide vote there keeps the compiler from overlapping the
         // rows' loads (measured on the logistic-regression step: 85.9 us without the vote, 88.7 with it), and in
         // the scans, whose tiles are loaded ahead in the same way (running sum of exp over 2^27 values: 210 against 268 us)
         << (e.g.kind == GroupKind::GEMM || e.g.kind == GroupKind::GEMV || e.g.kind == GroupKind::SCAN ? "#define GR_ANY_LANE(c) true\n#define GR_KEEP_BRANCH\n"
                                         : "#define GR_ANY_LANE(c) (__builtin_amdgcn_ballot_w64(c) != 0ull)\n#define GR_KEEP_BRANCH __builtin_amdgcn_sched_barrier(0)\n")
         << "static __device__ __forceinline__ float gr_maxf(float a, float b) { return (a >= b || a != a) ? a : b; }\n"
         "static __device__ __forceinline__ float gr_minf(float a, float b) { return (a <= b || a != a) ? a : b; }\n"
         // Correctly rounded square root in five instructions instead of the compiler's sixteen: the
         // hardware's reciprocal square root (1 ulp), then one Newton step on s = x*y with the residual
         // x - s*s taken exactly by an fma.  For every argument of magnitude 2^-96 or more, for zeros,
         // infinities, NaNs and negative numbers the result has the bits of the IEEE square root (all
         // 2^32 arguments are compared on the device by the test suite); below 2^-96 the residual would
         // underflow, so a wave in which any lane holds such an argument takes the library routine.
         // Zeros and infinity are put right by a select that only a wave holding an argument outside
         // [2^-96, inf) executes; other lanes of such a wave keep their value.
         "static __device__ __forceinline__ float gr_sqrtf(float x) {\n"
         "  const float y = __builtin_amdgcn_rsqf(x);\n"
         "  const float s = x * y, h = 0.5f * y;\n"
         "  float t = __builtin_fmaf(__builtin_fmaf(-s, s, x), h, s);\n"
         "  if (GR_ANY_LANE(!(x >= 0x1p-96f && x < __builtin_inff()))) {\n"
         "    GR_KEEP_BRANCH;\n"
         "    const bool tiny = __builtin_fabsf(x) < 0x1p-96f && x != 0.0f;\n"
         "    if (GR_ANY_LANE(tiny)) return sqrtf(x);\n"
         "    t = (x == 0.0f || x == __builtin_inff()) ? x : t;\n"
         "  }\n"
         "  return t;\n}\n"
         << kDeviceMath << "\n" << (calls(e.g, GR_TANH) || (e.g.pair && calls(*e.g.pair, GR_TANH)) ? std::string(kDeviceTanh) + "\n" : std::string()) <<
         "static __device__ __forceinline__ float gr_xor(float v, int m) { return __shfl_xor(v, m, 64); }\n"
         "static __device__ __forceinline__ int gr_xor(int v, int m) { return __shfl_xor(v, m, 64); }\n"
         "static __device__ __forceinline__ long long gr_xor(long long v, int m) {\n"
         "  int lo = __shfl_xor((int)(v & 0xffffffffll), m, 64), hi = __shfl_xor((int)(v >> 32), m, 64);\n"
         "  return ((long long)hi << 32) | (unsigned int)lo;\n}\n";
}

// Emits gr_comb<ph>(a, b) and the lane / block reduction helpers for a phase.
void phase_helpers(Em& e, int ph, int lanes) {
  const Phase& p = e.g.phases[ph];
  const char* T = cty(p.out_dtype);
  // combining two partial results never converts (unlike combining an element into an i64 sum)
  std::string comb;
  if (p.op == GR_SUM) comb = "(x + y)";
  else if (p.out_dtype == GR_F32) comb = std::string(p.op == GR_MAX ? "gr_maxf" : "gr_minf") + "(x, y)";
  else comb = std::string("(x ") + (p.op == GR_MAX ? ">=" : "<=") + " y ? x : y)";
  e.o << "static __device__ __forceinline__ " << T << " gr_comb" << ph << "(" << T << " x, " << T << " y) { return " << comb << "; }\n";
  int w = std::min(lanes, 64);
  e.o << "static __device__ __forceinline__ " << T << " gr_lanes" << ph << "(" << T << " v) {\n";
  for (int m = w / 2; m > 0; m >>= 1) e.o << "  v = gr_comb" << ph << "(v, gr_xor(v, " << m << "));\n";
  e.o << "  return v;\n}\n";
}

// ---- point program emission (scalar) -----------------------------------------

// Emits the instructions of `prog` needed for `want` as scalar statements.
// load_expr(instr) gives the expression of a LOAD; acc_expr the dot result.
void emit_scalar_program(Em& e, const std::vector<Instr>& prog, const std::vector<int>& want,
                         const std::function<std::string(const Instr&, int)>& load_expr, const std::string& acc_expr,
                         const std::string& prefix, const std::string& indent, std::vector<char>* done_io = nullptr) {
  std::vector<char> need(prog.size(), 0);
  std::vector<int> work(want);
  while (!work.empty()) {
    int i = work.back();
    work.pop_back();
    if (i < 0 || need[i]) continue;
    if (done_io && (*done_io)[i]) continue;
    need[i] = 1;
    if (prog[i].a >= 0) work.push_back(prog[i].a);
    if (prog[i].b >= 0) work.push_back(prog[i].b);
  }
  auto name = [&](int i) { return prefix + std::to_string(i); };
  for (size_t i = 0; i < prog.size(); ++i) {
    if (!need[i]) continue;
    const Instr& in = prog[i];
    e.o << indent << "const " << cty(in.dtype) << ' ' << name((int)i) << " = ";
    switch (in.kind) {
      case IKind::LOAD: e.o << load_expr(in, (int)i); break;
      case IKind::CONST: e.o << e.cst(in.cslot); break;
      case IKind::UNARY: e.o << Em::unop(in.op, in.dtype, name(in.a)); break;
      case IKind::BINARY:
        // a quotient whose divisor is a scalar constant of the program: the same in every lane
        if (in.op == GR_DIV && in.dtype == GR_F32 && in.b >= 0 && prog[in.b].kind == IKind::CONST) e.o << "gr_divc(" << name(in.a) << ", " << name(in.b) << ")";
        else e.o << Em::binop(in.op, in.dtype, name(in.a), name(in.b));
        break;
      case IKind::RED: e.o << "red" << in.phase; break;
      case IKind::ACC: e.o << acc_expr; break;
    }
    e.o << ";\n";
    if (done_io) (*done_io)[i] = 1;
  }
}

// Common kernel head: Args, extents.
void kernel_head(Em& e, const std::string& name, int threads = 256) {
  e.o << "extern \"C\" __global__ __launch_bounds__(" << threads << ") void " << name << "(Args a) {\n";
}

// Declares p<g>: pointer of each access group advanced by its base offset.
void group_pointers(Em& e, const std::string& indent, const std::vector<int>& skip = {}) {
  for (size_t gi = 0; gi < e.g.groups.size(); ++gi) {
    if (std::find(skip.begin(), skip.end(), (int)gi) != skip.end()) continue;
    const AccessGroup& ag = e.g.groups[gi];
    e.o << indent << "const GM " << cty(ag.dtype) << "* const " << e.qp << gi << " = (const GM " << cty(ag.dtype) << "*)" << e.slot(e.L.ptr[gi])
        << " + " << e.S(e.L.base[gi]) << ";\n";
  }
}

// ---- MAP ----------------------------------------------------------------------

void gen_map(Em& e) {
  const GroupPlan& g = e.g;
  const int rank = g.rank;
  const int TC = g.BX * 4 * g.UC, TR = g.BY * g.VR;
  const int cd = rank - 1, rd = rank - 2;
  prelude(e);
  kernel_head(e, kernel_name(g));
  e.o << "  const long long C = " << e.dim(cd) << ";\n";
  e.o << "  const long long R = " << (rank >= 2 ? e.dim(rd) : std::string("1")) << ";\n";
  if (g.flat == 1) e.o << "  const long long nvc = (C + 3) / 4, nrg = (R + " << g.VR - 1 << ") / " << g.VR << ";\n";
  // tile bookkeeping in 32-bit unsigned arithmetic (the grid has fewer than 2^31 tiles)
  else e.o << "  const unsigned nbx = (unsigned)((C + " << g.cphase + TC - 1 << ") / " << TC << "), nby = (unsigned)((R + " << TR - 1 << ") / " << TR << ");\n";
  e.o << "  unsigned tile = blockIdx.x;\n";
  if (g.xcd_remap) {
    // consecutive tiles go to the same XCD (workgroups are dealt round-robin over the 8 XCDs),
    // so tiles that share halo rows also share an L2
    e.o << "  { unsigned outer = 1;\n";
    for (int k = 0; k + 2 < rank; ++k) e.o << "    outer *= (unsigned)" << e.dim(k) << ";\n";
    e.o << "    const unsigned ntiles = " << (g.flat == 1 ? "(unsigned)((nvc * nrg * outer + 255) / 256)" : "nbx * nby * outer") << ", per = (ntiles + 7) / 8;\n"
           "    tile = (blockIdx.x % 8) * per + blockIdx.x / 8;\n"
           "    if (tile >= ntiles) return; }\n";
  }
  if (g.diag)
    // A transposed operand of a matrix whose rows are a power of two long: the tiles of one row
    // block lie megabytes apart in it, on few memory channels.  Workgroups in flight together
    // take different row blocks as well as different column blocks.  Column blocks next to each
    // other share cache lines of the output when its rows are not a multiple of 128 bytes long:
    // they go to the same XCD (workgroups are dealt round-robin over the 8 XCDs), whose L2 then
    // merges the two halves of such a line into one write.
    e.o << "  const unsigned slab = nbx * nby, olin = tile / slab, sl = tile % slab;\n"
           "  unsigned bx, by;\n"
           "  if ((nbx & 7) == 0) { const unsigned nq = nbx >> 3, l = sl >> 3; bx = (sl & 7) * nq + l % nq; by = (l / nq + bx) % nby; }\n"
           "  else { bx = sl % nbx; by = (sl / nbx + bx) % nby; }\n";
  else if (g.flat == 1) {
    // lanes in order over (outer index, row group, column group): no lane without a patch but the last workgroup's, and the
    // last group of columns (rows) starts four (VR) from the end, so that every patch lies inside the array
    e.o << "  long long frem = (long long)tile * 256 + threadIdx.x;\n  if (frem >= nvc * nrg";
    for (int k = 0; k + 2 < rank; ++k) e.o << " * " << e.dim(k);
    e.o << ") return;\n"
           "  const long long cg = gr_peel(frem, nvc), rg = gr_peel(frem, nrg);\n"
           "  const long long c0 = 4 * cg + 4 <= C ? 4 * cg : C - 4, r0 = " << g.VR << " * rg + " << g.VR << " <= R ? " << g.VR << " * rg : R - " << g.VR << ";\n";
  } else
    e.o << "  const unsigned bx = tile % nbx, t2 = tile / nbx, by = t2 % nby, olin = t2 / nby;\n";
  if (rank > 2) {
    e.o << "  unsigned orem = " << (g.flat == 1 ? "(unsigned)frem" : "olin") << ";\n";
    for (int k = rank - 3; k >= 0; --k) e.o << "  const long long i" << k << " = orem % (unsigned)" << e.dim(k) << "; orem /= (unsigned)" << e.dim(k) << ";\n";
  }
  if (g.flat != 1) {
    e.o << "  const int tx = threadIdx.x % " << g.BX << ", ty = threadIdx.x / " << g.BX << ";\n";
    const char* q = g.flat ? "q" : "";   // (of the tile; below: of a patch that lies inside the array)
    e.o << "  const long long r0" << q << " = (long long)by * " << TR << " + ty * " << g.VR << ", c0" << q << " = (long long)bx * " << TC << " + tx * 4" << (g.cphase ? " - " + std::to_string(g.cphase) : std::string()) << ";\n";
    if (g.flat)
      e.o << "  if (r0q >= R || c0q >= C) return;\n"
             "  const long long c0 = c0q + 4 <= C ? c0q : C - 4, r0 = r0q + " << g.VR << " <= R ? r0q : R - " << g.VR << ";\n";
  }
  group_pointers(e, "  ");
  for (size_t gi = 0; gi < g.groups.size(); ++gi) {
    const AccessGroup& ag = g.groups[gi];
    e.o << "  const GM " << cty(ag.dtype) << "* const p" << gi << " = q" << gi;
    for (int k = 0; k + 2 < rank; ++k) if (!ag.structural_zero[k]) e.o << " + i" << k << " * " << e.coef((int)gi, k);
    if (rank >= 2 && !ag.structural_zero[rd]) e.o << " + r0 * " << e.coef((int)gi, rd);
    char cc = access_class(ag, cd);
    if (cc == '1') e.o << " + c0";
    else if (cc == 'G') e.o << " + c0 * " << e.coef((int)gi, cd);
    e.o << ";\n";
  }
  // output strides are arguments: a C-contiguous result or the strided view of a slice assignment
  e.o << "  const long long oc = " << (g.out_unit ? std::string("1") : e.S(e.L.ocoef + cd)) << ", orow = " << (rank >= 2 ? e.S(e.L.ocoef + rd) : std::string("0")) << ";\n";
  e.o << "  GM " << cty(g.out_dtype) << "* const po = (GM " << cty(g.out_dtype) << "*)" << e.slot(e.L.out) << " + " << e.S(e.L.obase);
  for (int k = 0; k + 2 < rank; ++k) e.o << " + i" << k << " * " << e.S(e.L.ocoef + k);
  e.o << " + r0 * orow + c0 * oc;\n";

  // static part of a load's address: shifts times runtime coefficients
  auto shift_expr = [&](const Instr& in, bool with_col) {
    const AccessGroup& ag = g.groups[in.group];
    std::ostringstream s;
    bool any = false;
    for (int k = 0; k < rank; ++k) {
      if (in.delta[k] == 0 || ag.structural_zero[k]) continue;
      if (k == cd) {
        if (!with_col) continue;
        if (access_class(ag, cd) == '1') s << (any ? " + " : "") << in.delta[k];
        else s << (any ? " + " : "") << in.delta[k] << " * " << e.coef(in.group, k);
      } else s << (any ? " + " : "") << in.delta[k] << " * " << e.coef(in.group, k);
      any = true;
    }
    if (!any) s << "0";
    return s.str();
  };

  // ---- transposed operands: the workgroup's tile (64 columns by 64 or 128 rows) goes through LDS, loaded along the
  // operand's own contiguous dimension (the rows of the iteration space) ----
  if (g.stage_mask) {
    for (size_t gi = 0; gi < g.groups.size(); ++gi) {
      if (!(g.stage_mask >> gi & 1)) continue;
      const AccessGroup& ag = g.groups[gi];
      const char* T = cty(ag.dtype);
      const char* V4 = vty4(ag.dtype);
      // tile: 64 columns by STR = BY * VR rows of the iteration space, i.e. 64 runs of STR
      // contiguous elements of the operand
      const int STR = g.BY * g.VR, TPR = STR / 4, RPP = 256 / TPR, NPASS = 64 / RPP;
      // Row cc of the tile is rotated by 4 * (cc / 4) elements: a lane's four-element writes
      // (along the operand's contiguous dimension) and its four-element reads (rows of its patch,
      // one column) both touch every LDS bank once per eight lanes.
      const char* V4A = ag.dtype == GR_F32 ? "f4" : "i4";
      e.o << "  __shared__ __attribute__((aligned(16))) " << T << " tg" << gi << "[64][" << STR << "];\n";
      e.o << "  { const GM " << T << "* const pt = q" << gi;
      for (int k = 0; k + 2 < rank; ++k) if (!ag.structural_zero[k]) e.o << " + i" << k << " * " << e.coef((int)gi, k);
      e.o << " + (long long)by * " << STR << " + (long long)bx * 64 * " << e.coef((int)gi, cd) << ";\n";
      e.o << "    const int c1 = threadIdx.x / " << TPR << ", r4 = (threadIdx.x % " << TPR << ") * 4;\n";
      // interior tiles: every load is issued before the first LDS store
      e.o << "    if ((long long)bx * 64 + 64 <= C && (long long)by * " << STR << " + " << STR << " <= R) {\n"
             "      " << V4 << " w[" << NPASS << "];\n"
             "      _Pragma(\"unroll\") for (int i = 0; i < " << NPASS << "; ++i) w[i] = *(const GM " << V4 << "*)(pt + (c1 + " << RPP << " * i) * " << e.coef((int)gi, cd) << " + r4);\n"
             "      _Pragma(\"unroll\") for (int i = 0; i < " << NPASS << "; ++i) { const int cc = c1 + " << RPP << " * i;"
             " *(" << V4A << "*)&tg" << gi << "[cc][(r4 + 4 * (cc >> 2)) & " << STR - 1 << "] = w[i]; }\n"
             "    } else\n";
      e.o << "    for (int i = 0; i < " << NPASS << "; ++i) {\n      const int cc = c1 + " << RPP << " * i;\n"
             "      const long long gc = (long long)bx * 64 + cc, gr = (long long)by * " << STR << " + r4;\n"
             "      if (gc < C && gr + 4 <= R) { const " << V4 << " w = *(const GM " << V4 << "*)(pt + cc * " << e.coef((int)gi, cd) << " + r4);"
             " *(" << V4A << "*)&tg" << gi << "[cc][(r4 + 4 * (cc >> 2)) & " << STR - 1 << "] = w; }\n"
             "      else if (gc < C) { for (int j = 0; j < 4; ++j) if (gr + j < R) tg" << gi << "[cc][(r4 + j + 4 * (cc >> 2)) & " << STR - 1 << "] = pt[cc * " << e.coef((int)gi, cd) << " + r4 + j]; }\n"
             "    }\n  }\n";
    }
    e.o << "  __syncthreads();\n";
  }
  // ---- lanes whose whole patch lies inside the array: straight-line ----
  if (g.flat) e.o << "  {\n";
  else e.o << "  if (r0 + " << g.VR << " <= R && c0 + " << (g.UC - 1) * g.BX * 4 + 4 << " <= C" << (g.cphase ? " && c0 >= 0" : "") << ") {\n";
  // group the contiguous loads of the patch program into vector loads
  std::map<int, std::string> load_name;  // instr -> expression
  {
    // key: group + all deltas but the column one
    std::map<std::vector<int64_t>, std::vector<std::pair<int64_t, int>>> rows;
    std::vector<char> used(g.prog.size(), 0);
    {  // only loads reachable from the results
      std::vector<int> work(g.results.begin(), g.results.end());
      while (!work.empty()) {
        int i = work.back();
        work.pop_back();
        if (i < 0 || used[i]) continue;
        used[i] = 1;
        work.push_back(g.prog[i].a);
        work.push_back(g.prog[i].b);
      }
    }
    int nl = 0;
    std::set<std::string> staged_done;
    for (size_t i = 0; i < g.prog.size(); ++i) {
      const Instr& in = g.prog[i];
      if (in.kind != IKind::LOAD || !used[i]) continue;
      const AccessGroup& ag = g.groups[in.group];
      if (g.stage_mask >> in.group & 1) {
        // element (row r0 + dr, column c0 + dc) of the iteration space sits at [column][row] of the
        // tile (rotated): four rows of one column are one 16-byte LDS read
        const int dc = (int)in.delta[cd], dr = (int)in.delta[rd];
        const std::string nm = "S" + std::to_string(in.group) + "_" + std::to_string(dc) + "_" + std::to_string(dr / 4);
        if (staged_done.insert(nm).second)
          e.o << "    const " << (ag.dtype == GR_F32 ? "f4" : "i4") << ' ' << nm << " = *(const " << (ag.dtype == GR_F32 ? "f4" : "i4") << "*)&tg" << in.group
              << "[tx * 4 + " << dc << "][(ty * " << g.VR << " + " << dr / 4 * 4 << " + 4 * tx) & " << g.BY * g.VR - 1 << "];\n";
        load_name[(int)i] = nm + "[" + std::to_string(dr % 4) + "]";
        continue;
      }
      if (access_class(ag, cd) != '1') {
        load_name[(int)i] = "p" + std::to_string(in.group) + "[" + shift_expr(in, true) + "]";
        continue;
      }
      std::vector<int64_t> key{in.group};
      for (int k = 0; k < rank; ++k) if (k != cd) key.push_back(in.delta[k]);
      rows[key].push_back({in.delta[cd], (int)i});
    }
    for (auto& kv : rows) {
      auto& v = kv.second;
      std::sort(v.begin(), v.end());
      const Instr& first = g.prog[v[0].second];
      const AccessGroup& ag = g.groups[first.group];
      std::string rowoff = shift_expr(first, false);
      size_t i = 0;
      while (i < v.size()) {
        size_t run = 1;
        while (i + run < v.size() && v[i + run].first == v[i].first + (int64_t)run) ++run;
        size_t pos = 0;
        while (pos < run) {
          size_t take = run - pos >= 4 ? 4 : (run - pos >= 2 ? 2 : 1);
          int64_t dc = v[i + pos].first;
          std::string nm = "L" + std::to_string(nl++);
          std::string addr = "p" + std::to_string(first.group) + " + (" + rowoff + ") + " + std::to_string(dc);
          const char* lt = take == 4 ? vty4(ag.dtype) : (take == 2 ? vty2(ag.dtype) : cty(ag.dtype));
          e.o << "    const " << lt << ' ' << nm << " = " << e.ld(first.group, lt, addr) << ";\n";
          for (size_t q = 0; q < take; ++q)
            load_name[v[i + pos + q].second] = take == 1 ? nm : nm + "[" + std::to_string(q) + "]";
          pos += take;
        }
        i += run;
      }
    }
  }
  emit_scalar_program(e, g.prog, g.results,
                      [&](const Instr&, int id) { return load_name[id]; }, "0.0f", "t", "    ");
  {
    int ri = 0;
    for (int v = 0; v < g.VR; ++v)
      for (int u = 0; u < g.UC; ++u) {
        std::string off = std::to_string(v) + " * orow + " + std::to_string(u * g.BX * 4) + " * oc";
        if (g.out_dtype == GR_I64 || !g.out_unit) {
          for (int j = 0; j < 4; ++j) e.o << "    po[" << off << " + " << j << " * oc] = t" << g.results[ri + j] << ";\n";
        } else {
          const char* vt = g.out_dtype == GR_F32 ? "f4u" : "i4u";
          e.o << "    { " << vt << " ov; ov[0] = t" << g.results[ri] << "; ov[1] = t" << g.results[ri + 1] << "; ov[2] = t" << g.results[ri + 2]
              << "; ov[3] = t" << g.results[ri + 3] << "; " << ((g.nt & 8) ? "__builtin_nontemporal_store(ov, (GM " + std::string(vt) + "*)(po + " + off + "))" : "*(GM " + std::string(vt) + "*)(po + " + off + ") = ov") << "; }\n";
        }
        ri += 4;
      }
  }
  if (g.flat) { e.o << "  }\n}\n"; return; }
  // ---- narrow arrays: the lanes of the last, incomplete group of four columns (all rows of
  // their patch inside): the same patch program restricted to the columns that exist, scalar
  // loads and stores, no guards ----
  if (g.tail > 0) {
    e.o << "  } else if (r0 + " << g.VR << " <= R && c0 + " << g.tail << " == C) {\n";
    std::vector<int> want;
    for (int v = 0; v < g.VR; ++v)
      for (int j = 0; j < g.tail; ++j) want.push_back(g.results[(size_t)v * 4 + j]);
    emit_scalar_program(e, g.prog, want,
                        [&](const Instr& in, int) { return "p" + std::to_string(in.group) + "[" + shift_expr(in, true) + "]"; },
                        "0.0f", "w", "    ");
    for (int v = 0; v < g.VR; ++v)
      for (int j = 0; j < g.tail; ++j)
        e.o << "    po[" << v << " * orow + " << j << " * oc] = w" << g.results[(size_t)v * 4 + j] << ";\n";
  }
  // ---- lanes on the array's edge: one guarded point at a time ----
  e.o << "  } else {\n"
         "    for (int v = 0; v < " << g.VR << "; ++v)\n"
         "      for (int u = 0; u < " << g.UC << "; ++u)\n"
         "        for (int j = 0; j < 4; ++j) {\n"
         "          const long long cj = (long long)u * " << g.BX * 4 << " + j;\n"
         "          if (r0 + v < R && c0 + cj < C" << (g.cphase ? " && c0 + cj >= 0" : "") << ") {\n";
  emit_scalar_program(e, g.prog1, {g.result1},
                      [&](const Instr& in, int) {
                        const AccessGroup& ag = g.groups[in.group];
                        std::string s = "p" + std::to_string(in.group) + "[" + shift_expr(in, true);
                        if (rank >= 2 && !ag.structural_zero[rd]) s += " + v * " + e.coef(in.group, rd);
                        char cc = access_class(ag, cd);
                        if (cc == '1') s += " + cj";
                        else if (cc == 'G') s += " + cj * " + e.coef(in.group, cd);
                        return s + "]";
                      },
                      "0.0f", "s", "            ");
  e.o << "            po[v * orow + cj * oc] = s" << g.result1 << ";\n"
         "          }\n        }\n  }\n}\n";
}

// A map that writes the array it reads at positions a few rows and columns away.  A workgroup loads all that its
// tile needs, waits until all of its waves have, and only then stores.  The cells around a tile, which other workgroups write:
//
// - Many tiles: they come from copies that gr_map_save made in a launch before: whole rows above and below every row of tiles, and a
//   few columns on either side of every boundary between tiles of a row.  Bound by HBM or the caches: 2 rows saved, and read again, per VR
//   rows read and written.
//
// - Few tiles (in_place_once): one launch.  A workgroup marks its tile as loaded and looks at the marks of the tiles around it until they
//   are loaded too.  It does not look more often than `polls` times, because a tile that it waits for may not have been started: then it
//   saves the cells of its own tile that others read (while they are still the old ones), marks the tile as saved, and stores.  A workgroup
//   that finds a tile beside it saved takes the cells there from what was saved; whatever it loaded itself, before it looked, from a tile
//   that was not marked so is old, since marks precede stores.  So no workgroup depends on another one's progress.  Marks carry the number
//   of the launch; they and saved cells are written with relaxed agent-scope atomics that have completed (vmcnt) before what they precede
//   is issued.  Bound by launches: ten sweeps of 1000^2 72 -> 68 us, 4535 x 400 101 -> 88, 100 x 300 97 -> 60 by one launch instead of two;
//   with more tiles than are there at a time the marks' round trips hold the chip's workgroups: 2300^2 129 -> 142, 4096^2 279 -> 369.
void gen_map_in_place(Em& e) {
  const GroupPlan& g = e.g;
  const int TC = g.BX * 4, TR = g.BY * g.VR, HT = g.halo[0], HB = g.halo[1], HL = g.halo[2], HR = g.halo[3];
  const int off = (HL + 3) / 4 * 4, offr = (HR + 3) / 4 * 4;
  std::ostream& o = e.o;
  const std::string T = cty(g.out_dtype), V4 = vty4(g.out_dtype), V2 = vty2(g.out_dtype);
  const bool once = g.in_place_once;
  const int PT = in_place_saved(g);   // saved cells per tile
  prelude(e);
  if (once) {
    auto head = [&](const char* name) {
      kernel_head(e, name);
      o << "  const int C = (int)" << e.dim(1) << ", R = (int)" << e.dim(0) << ", nbx = (C + " << g.cphase + TC - 1 << ") / " << TC << ", nby = (R + " << TR - 1 << ") / " << TR << ";\n"
           "  GM unsigned long long* const marks = (GM unsigned long long*)" << e.slot(e.L.extra + 1) << ";\n";
    };
    head("gr_map_clear");
    o << "  const unsigned i = blockIdx.x * 256 + threadIdx.x;\n  if (i < (unsigned)(nbx * nby)) marks[i] = 0ull;\n}\n";
    head(kernel_name(g).c_str());
    o << "  const long long orow = " << e.S(e.L.ocoef) << ";\n"
         "  GM " << T << "* const po = (GM " << T << "*)" << e.slot(e.L.out) << " + " << e.S(e.L.obase) << ";\n"
         "  GM " << T << "* const saved = (GM " << T << "*)" << e.slot(e.L.extra) << ";\n"
         "  const unsigned long long TAG = " << e.slot(e.L.extra + 2) << " << 32;\n  unsigned polls = (unsigned)(" << e.slot(e.L.extra + 2) << " >> 32);\n";
  } else {
    auto head = [&](const char* name) {
      kernel_head(e, name);
      o << "  const int C = (int)" << e.dim(1) << ", R = (int)" << e.dim(0) << ", nbx = (C + " << g.cphase + TC - 1 << ") / " << TC << ", nby = (R + " << TR - 1 << ") / " << TR << ";\n"
           "  const long long orow = " << e.S(e.L.ocoef) << ", pitch = (long long)nbx * " << TC + 0 << " + " << off + offr << ";\n"
           "  GM " << T << "* const po = (GM " << T << "*)" << e.slot(e.L.out) << " + " << e.S(e.L.obase) << ";\n"
           "  GM " << T << "* const rows = (GM " << T << "*)" << e.slot(e.L.extra) << ";\n"
           "  GM " << T << "* const cols = rows + (long long)nby * " << HT + HB << " * pitch;\n  (void)cols; (void)pitch;\n";
    };
    head("gr_map_save");
    o << "  unsigned idx = blockIdx.x * 256 + threadIdx.x;\n  const unsigned quads = (unsigned)(pitch / 4), first = quads * (unsigned)nby * " << HT + HB << "u;\n"
         "  if (idx < first) {\n"
         "    const int i4 = (int)(idx % quads), line = (int)(idx / quads), h = line % " << std::max(1, HT + HB) << ", by = line / " << std::max(1, HT + HB) << ";\n"
         "    const int at = h < " << HT << " ? by * " << TR << " - " << HT << " + h : by * " << TR << " + " << TR - HT << " + h, r = at < R + " << HB - 1 << " ? at : R + " << HB - 1 << ";\n"
         "    const int c = 4 * i4 - " << off + g.cphase << ";\n"
         "    GM " << T << "* const to = rows + (long long)line * pitch + 4 * i4;\n    const GM " << T << "* const from = po + r * orow;\n"
         "    if (c >= " << -HL << " && c + 4 <= C + " << HR << ") *(GM " << V4 << "*)to = *(const GM " << V4 << "*)(from + c);\n"
         "    else for (int j = 0; j < 4; ++j) { const int k = c + j; to[j] = from[k < " << -HL << " ? " << -HL << " : (k < C + " << HR << " ? k : C + " << HR - 1 << ")]; }\n"
         "    return;\n  }\n";
    if (HL + HR > 0)
      o << "  idx -= first;\n  const unsigned lines = (unsigned)R + " << HT + HB << "u;\n"
           "  if (idx >= lines * (unsigned)(nbx - 1) * " << HL + HR << "u) return;\n"
           "  const int q = (int)(idx % " << HL + HR << "), line = (int)(idx / " << HL + HR << "), r = (int)(line % lines) - " << HT << ", b = (int)(line / lines);\n"
           // (a boundary near the end of the rows: columns that no element reads are not there)
           "  const int c = (b + 1) * " << TC << " - " << g.cphase << " + q - " << HL << ";\n"
           "  cols[idx] = po[r * orow + (c < C + " << HR << " ? c : C + " << HR - 1 << ")];\n";
    o << "}\n";
    head(kernel_name(g).c_str());
  }
  o << "  const unsigned ntiles = (unsigned)(nbx * nby), per = (ntiles + 7) / 8, tile = (blockIdx.x % 8) * per + blockIdx.x / 8;\n"
       "  if (blockIdx.x / 8 >= per || tile >= ntiles) return;\n"
       "  const int bx = (int)(tile % (unsigned)nbx), by = (int)(tile / (unsigned)nbx), tx = threadIdx.x % " << g.BX << ", ty = " << (g.BY > 1 ? "threadIdx.x / " + std::to_string(g.BX) : std::string("0")) << ";\n"
       "  const int r0 = by * " << TR << " + ty * " << g.VR << ", c0 = bx * " << TC << " + tx * 4 - " << g.cphase << ", rmax = R + " << HB - 1 << ";\n"
       "  const bool live = c0 < C, whole = c0 >= 0 && c0 + 4 <= C;\n  (void)ty;\n";
  int self = -1;
  for (size_t i = 0; i < g.groups.size(); ++i) if (!g.groups[i].structural_zero[0] || !g.groups[i].structural_zero[1]) self = (int)i;
  for (size_t i = 0; i < g.groups.size(); ++i)
    if ((int)i != self) o << "  const GM " << cty(g.groups[i].dtype) << "* const q" << i << " = (const GM " << cty(g.groups[i].dtype) << "*)" << e.slot(e.L.ptr[i]) << " + " << e.S(e.L.base[i]) << ";\n";
  // loads of the patch: per row (relative to r0) the columns (relative to c0)
  std::vector<char> used(g.prog.size(), 0);
  std::vector<int> work(g.results.begin(), g.results.end());
  while (!work.empty()) {
    const int i = work.back();
    work.pop_back();
    if (i < 0 || used[i]) continue;
    used[i] = 1;
    work.push_back(g.prog[i].a);
    work.push_back(g.prog[i].b);
  }
  std::map<int, std::map<int, int>> at;   // row -> column -> instruction
  std::map<int, std::string> name;
  for (size_t i = 0; i < g.prog.size(); ++i) {
    const Instr& in = g.prog[i];
    if (in.kind != IKind::LOAD || !used[i]) continue;
    if (in.group != self) name[(int)i] = "q" + std::to_string(in.group) + "[0]";
    else at[(int)in.delta[0] + g.self_row][(int)in.delta[1] + g.self_col] = (int)i;
  }
  auto rn = [](int s) { return s < 0 ? "m" + std::to_string(-s) : std::to_string(s); };
  std::ostringstream fast, slow, left, right, again;
  std::set<int> edge;
  bool reads[3][3] = {};   // tiles around it that a tile reads
  int nl = 0;
  for (const auto& row : at) {
    const int s = row.first;
    const std::string grid = "po + (long long)(r0 + " + std::to_string(s) + " < rmax ? r0 + " + std::to_string(s) + " : rmax) * orow + c0";
    const int h = s < 0 ? HT + s : HT + s - g.VR;
    const std::string saved = "rows + (by * " + std::to_string(HT + HB) + "ll + " + std::to_string(h) + ") * pitch + (c0 + " + std::to_string(off + g.cphase) + ")";
    const std::string w = "w" + rn(s);
    o << "  const GM " << T << "* const " << w << " = ";
    if (once || (s >= 0 && s < g.VR)) o << grid;
    else if (g.BY == 1) o << saved;
    else o << (s < 0 ? "ty == 0" : "ty == " + std::to_string(g.BY - 1)) << " ? (const GM " << T << "*)(" << saved << ") : (const GM " << T << "*)(" << grid << ")";
    o << ";\n";
    std::vector<std::pair<int, int>> v(row.second.begin(), row.second.end());
    size_t i = 0;
    while (i < v.size()) {
      size_t run = 1;
      while (i + run < v.size() && v[i + run].first == v[i].first + (int)run) ++run;
      for (size_t pos = 0; pos < run;) {
        const size_t take = run - pos >= 4 ? 4 : (run - pos >= 2 ? 2 : 1);
        const int dc = v[i + pos].first;
        const std::string nm = "L" + std::to_string(nl++), ty = take == 4 ? V4 : (take == 2 ? V2 : T);
        o << "  " << ty << ' ' << nm << ";\n";
        fast << "    " << nm << " = *(const GM " << ty << "*)(" << w << " + " << dc << ");\n";
        for (size_t q = 0; q < take; ++q) {
          const int c = dc + (int)q;
          const std::string el = take == 1 ? nm : nm + "[" + std::to_string(q) + "]";
          name[v[i + pos + q].second] = el;
          edge.insert(c);
          slow << "    " << el << " = " << w << "[k" << rn(c) << "];\n";
          const int dy = s < 0 ? 0 : (s >= g.VR ? 2 : 1), dx = c < 0 ? 0 : (c >= 4 ? 2 : 1);
          if (dy != 1 || dx != 1) {
            reads[dy][1] = reads[dy][1] || dy != 1;
            reads[1][dx] = reads[1][dx] || dx != 1;
            reads[dy][dx] = true;
            again << "    " << el << " = fetch(r0 + " << s << ", c0 + " << c << ", " << el << ");\n";
          }
          const std::string line = "[(r0 + " + std::to_string(s) + " < rmax ? r0 + " + std::to_string(s) + " : rmax) * " + std::to_string(HL + HR) + "ll + ";
          if (c < 0) left << "    " << el << " = cb" << line << HL + c << "];\n";
          if (c >= 4) right << "    " << el << " = cb" << line << HL + c - 4 << "];\n";
        }
        pos += take;
      }
      i += run;
    }
  }
  o << "  if (whole) {\n" << fast.str() << "  } else if (live) {\n";
  for (int c : edge) o << "    const int k" << rn(c) << " = (c0 + " << c << " < " << -HL << " ? " << -HL << " : (c0 + " << c << " < C + " << HR << " ? c0 + " << c << " : C + " << HR - 1 << ")) - c0;\n";
  o << slow.str() << "  }\n";
  const std::string cb = "    const GM " + T + "* const cb = cols + ((long long)";
  if (HL > 0 && !once) o << "  if (tx == 0 && bx > 0) {\n" << cb << "(bx - 1) * (R + " << HT + HB << ") + " << HT << ") * " << HL + HR << ";\n" << left.str() << "  }\n";
  if (HR > 0 && !once) o << "  if (tx == " << g.BX - 1 << " && bx + 1 < nbx && live) {\n" << cb << "bx * (R + " << HT + HB << ") + " << HT << ") * " << HL + HR << ";\n" << right.str() << "  }\n";
  // every load of the workgroup has returned before any of its stores is issued
  o << "  asm volatile(\"s_waitcnt vmcnt(0)\" ::: \"memory\");\n  __syncthreads();\n";
  if (once) {
    o << "  __shared__ unsigned near[9];\n"
         "  if (threadIdx.x == 0) __hip_atomic_store((unsigned long long*)&marks[tile], TAG | 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);\n"
         "  if (threadIdx.x < 9) {\n"
         "    const int y = by + (int)threadIdx.x / 3 - 1, x = bx + (int)threadIdx.x % 3 - 1;\n    unsigned state = 1;\n    constexpr unsigned around = ";
    unsigned around = 0;   // tiles that it reads, or that read it
    for (int dy = 0; dy < 3; ++dy) for (int dx = 0; dx < 3; ++dx) if (reads[dy][dx]) around |= 1u << (dy * 3 + dx) | 1u << (8 - dy * 3 - dx);
    o << around << "u;\n"
         "    if ((around >> threadIdx.x & 1) && x >= 0 && x < nbx && y >= 0 && y < nby)\n"
         "      for (;;) {\n        const unsigned long long w = __hip_atomic_load((unsigned long long*)&marks[y * nbx + x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);\n"
         "        state = (w ^ TAG) >> 32 ? 0u : (unsigned)w;\n        if (state || !polls) break;\n        --polls;\n        __builtin_amdgcn_s_sleep(1);\n      }\n"
         "    near[threadIdx.x] = state;\n  }\n  __syncthreads();\n"
         "  bool waited = true, old = false;\n"
         "#pragma unroll\n  for (int q = 0; q < 9; ++q) { waited = waited && near[q] != 0; old = old || near[q] == 2; }\n"
         "  if (!waited) {\n"
         "    GM unsigned* const to = (GM unsigned*)saved + (long long)tile * " << PT << ";\n"
         "    for (int i = threadIdx.x; i < " << (HT + HB) * TC << "; i += 256) {\n"
         "      const int h = i / " << TC << ", r = by * " << TR << " + (h < " << HT << " ? " << TR - HT << " + h : h - " << HT << "), c = bx * " << TC << " - " << g.cphase << " + i % " << TC << ";\n"
         "      if (r < R && c >= 0 && c < C) __hip_atomic_store((unsigned*)(to + i), *(const GM unsigned*)(po + r * orow + c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);\n    }\n";
    if (HL + HR > 0)
      o << "    for (int i = threadIdx.x; i < " << (HL + HR) * TR << "; i += 256) {\n"
           "      const int q = i % " << HL + HR << ", r = by * " << TR << " + i / " << HL + HR << ", c = bx * " << TC << " - " << g.cphase << " + (q < " << HL << " ? " << TC - HL << " + q : q - " << HL << ");\n"
           "      if (r < R && c >= 0 && c < C) __hip_atomic_store((unsigned*)(to + " << (HT + HB) * TC << " + i), *(const GM unsigned*)(po + r * orow + c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);\n    }\n";
    o << "    asm volatile(\"s_waitcnt vmcnt(0)\" ::: \"memory\");\n    __syncthreads();\n"
         "    if (threadIdx.x == 0) {\n      __hip_atomic_store((unsigned long long*)&marks[tile], TAG | 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);\n"
         "      asm volatile(\"s_waitcnt vmcnt(0)\" ::: \"memory\");\n    }\n    __syncthreads();\n  }\n"
         "  if (!live) return;\n"
         "  if (old) {\n"
         "    auto fetch = [&](int r, int c, " << T << " v) -> " << T << " {\n"
         "      if (r < 0 || r >= R || c < 0 || c >= C) return v;\n"
         "      const int y = r / " << TR << ", x = (c + " << g.cphase << ") / " << TC << ", dy = y - by, dx = x - bx;\n"
         "      if (near[4 + 3 * dy + dx] != 2) return v;\n"
         "      const int lr = r - y * " << TR << ", lc = c + " << g.cphase << " - x * " << TC << ";\n"
         "      const int at = dy != 0 ? (dy < 0 ? lr - " << TR - HT << " : " << HT << " + lr) * " << TC << " + lc : " << (HT + HB) * TC << " + lr * " << HL + HR << " + (dx < 0 ? lc - " << TC - HL << " : " << HL << " + lc);\n"
         "      const unsigned w = __hip_atomic_load((unsigned*)saved + (long long)(y * nbx + x) * " << PT << " + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);\n"
         "      return " << (g.out_dtype == GR_F32 ? "__uint_as_float(w)" : "(int)w") << ";\n    };\n"
      << again.str() << "  }\n";
  } else o << "  if (!live) return;\n";
  emit_scalar_program(e, g.prog, g.results, [&](const Instr&, int id) { return name[id]; }, "0", "t", "  ");
  for (int v = 0; v < g.VR; ++v) {
    const int* t = &g.results[(size_t)v * 4];
    o << "  if (r0 + " << v << " < R) {\n    GM " << T << "* const to = po + (r0 + " << v << ") * orow + c0;\n"
         "    if (whole) { " << V4 << " ov; ov[0] = t" << t[0] << "; ov[1] = t" << t[1] << "; ov[2] = t" << t[2] << "; ov[3] = t" << t[3] << "; *(GM " << V4 << "*)to = ov; }\n    else {\n";
    for (int j = 0; j < 4; ++j) o << "      if (c0 + " << j << " >= 0 && c0 + " << j << " < C) to[" << j << "] = t" << t[j] << ";\n";
    o << "    }\n  }\n";
  }
  o << "}\n";
}

// ---- ROWRED -------------------------------------------------------------------

// Short rows whose elements come from pairs of operands, one that follows the first kept dimension
// and one that follows the second (points and centres: sum over k of f(P[m,k], C[n,k])), one value
// per row.  A lane keeps the K elements of its own operand's row in registers and walks the other
// operand's rows, whose elements are the same for all lanes and come through the scalar unit; the
// groups of lanes of the general kernel load both elements of every pair instead.  Bound by vector
// issue.  The elements of a row are combined in the order in which the general kernel's lanes
// (and the interpreter's) combine them: four in turn per lane, lanes in a butterfly.
void gen_rowred_pairs(Em& e) {
  const GroupPlan& g = e.g;
  const int ld = g.pair_lane, ud = 1 - ld, K = g.pair_k, RT = g.row_threads, UJ = 4;
  const Phase& ph = g.phases[0];
  const std::string T = cty(ph.out_dtype);
  prelude(e);
  phase_helpers(e, 0, RT);
  e.o << "#define CM __attribute__((address_space(4)))\n";
  kernel_head(e, kernel_name(g));
  // (results of a lane are neighbours in the output: they pass through LDS, so that a wave's stores cover whole runs of it)
  const bool turn = ud == 1 && g.out_dtype != GR_I64;
  const char* OT = cty(g.out_dtype);
  const char* OV = g.out_dtype == GR_F32 ? "f4" : "i4";
  // Workgroups of the same 256 rows, which write neighbouring pieces of the same output rows, share an XCD (8 of them, dealt in
  // turn).  Fewer than 16 blocks of 256 rows are dealt without that: XCDs would be left without work (of 4 blocks half of them:
  // 1000 x 1000 squared distances in 16 dimensions 6.6 -> 5.4 us, in 32 12.2 -> 8.4; of 12 a quarter, 3000 x 2000 x 32 20.2 -> 18.5;
  // of 20 blocks the sharing is worth more, 5000 x 64 x 32 4.8 against 5.3).
  e.o << "  const long long NL = " << e.dim(ld) << ", NU = " << e.dim(ud) << ", CH = " << e.S(e.L.extra) << ";\n"
         "  const unsigned NUB = (unsigned)" << e.S(e.L.extra + 1) << ", NLB = (unsigned)((NL + 255) / 256), GRP = NLB < " << kPairSpread << " ? NLB : 8, set = blockIdx.x / (GRP * NUB), in_set = blockIdx.x % (GRP * NUB);\n"
         "  const long long lbeg = (long long)(set * GRP + in_set % GRP) * 256, lraw = lbeg + threadIdx.x, ubeg = in_set / GRP * CH, uend = ubeg + CH < NU ? ubeg + CH : NU;\n"
         "  if (lbeg >= NL || ubeg >= NU) return;\n"
         "  const bool ok = lraw < NL;\n"
         "  const long long lane = ok ? lraw : NL - 1;\n";
  if (turn) e.o << "  __shared__ __attribute__((aligned(16))) " << OT << " sm[256][" << kPairBlock + 4 << "];\n";   // (this pitch: four-element writes and reads without bank conflicts)
  std::vector<char> in_value(g.prog.size(), 0);
  {
    std::vector<int> work{ph.value};
    while (!work.empty()) {
      const int i = work.back();
      work.pop_back();
      if (i < 0 || in_value[i]) continue;
      in_value[i] = 1;
      work.push_back(g.prog[i].a);
      work.push_back(g.prog[i].b);
    }
  }
  auto kexpr = [&](const Instr& in, int k) -> std::string {
    const AccessGroup& ag = g.groups[in.group];
    if (ag.structural_zero[2]) return "0";
    if (access_class(ag, 2) == '1') return std::to_string(k + in.delta[2]);
    return std::to_string(k + in.delta[2]) + " * " + e.coef(in.group, 2);
  };
  // the lane's own operand elements
  for (size_t i = 0; i < g.prog.size(); ++i) {
    const Instr& in = g.prog[i];
    if (in.kind != IKind::LOAD || !in_value[i]) continue;
    const AccessGroup& ag = g.groups[in.group];
    if (ag.structural_zero[ld]) continue;
    const std::string id = std::to_string(i);
    e.o << "  const GM " << cty(in.dtype) << "* const pl" << id << " = (const GM " << cty(in.dtype) << "*)" << e.slot(e.L.ptr[in.group]) << " + " << e.S(e.L.base[in.group])
        << " + (lane + " << in.delta[ld] << ") * " << e.coef(in.group, ld) << ";\n";
    if (ag.structural_zero[2]) { e.o << "  const " << cty(in.dtype) << " x" << id << "_0 = pl" << id << "[0];\n"; continue; }
    int k = 0;
    if (access_class(ag, 2) == '1')
      for (; k + 4 <= K; k += 4) {
        e.o << "  const " << vty4(in.dtype) << " xv" << id << "_" << k << " = *(const GM " << vty4(in.dtype) << "*)(pl" << id << " + " << kexpr(in, k) << ");\n";
        for (int j = 0; j < 4; ++j) e.o << "  const " << cty(in.dtype) << " x" << id << "_" << k + j << " = xv" << id << "_" << k << "[" << j << "];\n";
      }
    for (; k < K; ++k) e.o << "  const " << cty(in.dtype) << " x" << id << "_" << k << " = pl" << id << "[" << kexpr(in, k) << "];\n";
  }
  e.o << "  GM " << cty(g.out_dtype) << "* const out = (GM " << cty(g.out_dtype) << "*)" << e.slot(e.L.out) << ";\n";
  e.o << "  for (long long u0 = ubeg; u0 < uend; u0 += " << UJ << ") {\n";
  for (int j = 0; j < UJ; ++j) {
    e.o << "    const long long u_" << j << " = u0 + " << j << " < NU ? u0 + " << j << " : NU - 1;\n    (void)u_" << j << ";\n";
    for (size_t i = 0; i < g.prog.size(); ++i) {
      const Instr& in = g.prog[i];
      if (in.kind != IKind::LOAD || !in_value[i] || !g.groups[in.group].structural_zero[ld]) continue;
      e.o << "    const CM " << cty(in.dtype) << "* const pu" << i << "_" << j << " = (const CM " << cty(in.dtype) << "*)(" << e.slot(e.L.ptr[in.group]) << " + 4 * (" << e.S(e.L.base[in.group]);
      if (!g.groups[in.group].structural_zero[ud]) e.o << " + (u_" << j << " + " << in.delta[ud] << ") * " << e.coef(in.group, ud);
      e.o << "));\n";
    }
  }
  const int summed = square_root_of(g, 0) >= 0 ? square_root_of(g, 0) : ph.value;
  // leaves of the butterfly in the order in which lane 0 meets them, the rows of UJ results side by side
  int next = 0;
  std::function<int(int, int)> tree = [&](int off, int stride) -> int {
    const int me = next++;
    if (stride == RT) {
      for (int j = 0; j < UJ; ++j) {
        const std::string acc = "t" + std::to_string(me) + "_" + std::to_string(j);
        e.o << "    " << T << " " << acc << " = " << Em::identity(ph) << ";\n";
        for (int q = 0; q < 4 && 4 * off + q < K; ++q) {
          const int k = 4 * off + q;
          e.o << "    {\n";
          emit_scalar_program(e, g.prog, {summed},
                              [&](const Instr& in, int id) -> std::string {
                                const AccessGroup& ag = g.groups[in.group];
                                if (!ag.structural_zero[ld]) return "x" + std::to_string(id) + "_" + std::to_string(ag.structural_zero[2] ? 0 : k);
                                return "pu" + std::to_string(id) + "_" + std::to_string(j) + "[" + kexpr(in, k) + "]";
                              },
                              "0.0f", "v", "      ");
          e.o << "      " << acc << " = " << Em::accumulate(g, 0, acc, [](int i) { return "v" + std::to_string(i); }) << ";\n    }\n";
        }
      }
      return me;
    }
    const int a = tree(off, 2 * stride), b = tree(off + stride, 2 * stride);
    for (int j = 0; j < UJ; ++j)
      e.o << "    const " << T << " t" << me << "_" << j << " = gr_comb0(t" << a << "_" << j << ", t" << b << "_" << j << ");\n";
    return me;
  };
  const int top = tree(0, 1);
  const char* const at[2] = {ld == 0 ? "lane" : "u_", ld == 0 ? "u_" : "lane"};
  for (int j = 0; j < UJ; ++j) {
    const std::string sj = std::to_string(j);
    e.o << "    " << cty(g.out_dtype) << " o" << j << ";\n    {\n      const " << T << " red0 = t" << top << "_" << j << "; (void)red0;\n";
    emit_scalar_program(e, g.prog, {g.results[0]},
                        [&](const Instr& in, int) -> std::string {
                          const AccessGroup& ag = g.groups[in.group];
                          std::string p = "((const GM " + std::string(cty(in.dtype)) + "*)" + e.slot(e.L.ptr[in.group]) + " + " + e.S(e.L.base[in.group]);
                          for (int d = 0; d < 2; ++d)
                            if (!ag.structural_zero[d]) p += " + (" + std::string(at[d]) + (d == ud ? sj : "") + " + " + std::to_string(in.delta[d]) + ") * " + e.coef(in.group, d);
                          return p + ")[0]";
                        },
                        "0.0f", "w", "      ");
    e.o << "      o" << j << " = w" << g.results[0] << ";\n    }\n";
  }
  if (turn) {
    e.o << "    { " << OV << " ov; ov[0] = o0; ov[1] = o1; ov[2] = o2; ov[3] = o3; *(" << OV << "*)&sm[threadIdx.x][u0 - ubeg] = ov; }\n  }\n"
           "  __syncthreads();\n"
           "  const unsigned nu = (unsigned)(uend - ubeg), lpr = (nu + 3) / 4, step = 256 / lpr, c4 = threadIdx.x % lpr * 4;\n"
           "  if (threadIdx.x >= step * lpr) return;\n"
           "  for (unsigned r = threadIdx.x / lpr; r < 256 && lbeg + r < NL; r += step) {\n"
           "    const " << OV << " ov = *(const " << OV << "*)&sm[r][c4];\n"
           "    GM " << OT << "* const po = out + (lbeg + r) * NU + ubeg + c4;\n"
           "    if (c4 + 4 <= nu) *(GM " << OV << "u*)po = ov;\n"
           "    else { po[0] = ov[0]; if (c4 + 1 < nu) po[1] = ov[1]; if (c4 + 2 < nu) po[2] = ov[2]; }\n"
           "  }\n}\n";
    return;
  }
  e.o << "    if (ok) {\n";
  for (int j = 0; j < UJ; ++j) {
    if (ud == 1) e.o << "      if (u0 + " << j << " < uend) out[lane * NU + u0 + " << j << "] = o" << j << ";\n";
    else e.o << "      if (u0 + " << j << " < uend) out[(u0 + " << j << ") * NL + lane] = o" << j << ";\n";
  }
  e.o << "    }\n  }\n}\n";
}

void gen_rowred(Em& e) {
  const GroupPlan& g = e.g;
  if (g.pair_k) { gen_rowred_pairs(e); return; }
  const int rank = g.rank, cd = rank - 1;
  const int RT = g.row_threads, NP = g.NP, BT = std::max(256, RT), RB = BT / RT;
  const int nph = (int)g.phases.size();
  prelude(e);
  for (int ph = 0; ph < nph; ++ph) phase_helpers(e, ph, RT);

  // stage of first computation and liveness across stages
  const int nstage = nph + 1;
  std::vector<int> stage_of(g.prog.size(), -1);
  std::vector<std::vector<int>> stage_instrs(nstage);
  std::vector<char> keep(g.prog.size(), 0);
  for (int s = 0; s < nstage; ++s) {
    int want = s < nph ? g.phases[s].value : (g.results.empty() ? -1 : g.results[0]);
    std::vector<int> work{want};
    std::vector<char> seen(g.prog.size(), 0);
    while (!work.empty()) {
      int i = work.back();
      work.pop_back();
      if (i < 0 || seen[i]) continue;
      seen[i] = 1;
      if (stage_of[i] >= 0 && stage_of[i] < s) { keep[i] = 1; continue; }
      stage_of[i] = s;
      work.push_back(g.prog[i].a);
      work.push_back(g.prog[i].b);
    }
    for (size_t i = 0; i < g.prog.size(); ++i) if (stage_of[i] == s) stage_instrs[s].push_back((int)i);
  }

  kernel_head(e, kernel_name(g), BT);
  e.o << "  const long long C = " << e.dim(cd) << ";\n  long long ROWS = 1;\n";
  for (int k = 0; k < cd; ++k) e.o << "  ROWS *= " << e.dim(k) << ";\n";
  e.o << "  const int lane = threadIdx.x % " << RT << ";\n";
  // several rows per lane group (short rows, one value per row): the per-row code below is written
  // once into `body` and placed in two loops, see the end of this function
  const int RPT = (g.row_iters > 1 && RT <= 64 && g.out_per_row) ? g.row_iters : 1;
  // exact: the row is exactly as wide as the lanes' positions, no column guards anywhere
  auto emit_body = [&](bool exact) {
  if (RPT > 1) {
    e.o << "      const long long row = ((long long)blockIdx.x * " << RPT << " + rr) * " << RB << " + threadIdx.x / " << RT << ";\n      const bool row_ok = true;\n";
  } else if (RT <= 64) {
    // no workgroup barrier in this variant: lanes of rows past the end simply leave
    e.o << "  const long long row = (long long)blockIdx.x * " << RB << " + threadIdx.x / " << RT << ";\n";
    e.o << "  if (row >= ROWS) return;\n  const bool row_ok = true;\n";
  } else {
    // rows span several waves and combine through LDS behind a barrier every wave reaches:
    // lanes of a row past the end recompute the last row and skip the stores
    e.o << "  const long long row_raw = (long long)blockIdx.x * " << RB << " + threadIdx.x / " << RT << ";\n";
    e.o << "  const bool row_ok = row_raw < ROWS;\n  const long long row = row_ok ? row_raw : ROWS - 1;\n";
    e.o << "  __shared__ long long gr_sm[" << std::max(nph, 1) << "][" << BT / 64 << "];\n";
  }
  e.o << "  (void)row_ok;\n";
  if (cd >= 1) {
    e.o << "  long long rrem = row;\n";
    for (int k = cd - 1; k >= 0; --k) {
      if (k == 0) e.o << "  const long long i0 = rrem;\n";  // what is left is below the outermost extent
      else e.o << "  const long long i" << k << " = gr_peel(rrem, " << e.dim(k) << ");\n";
    }
  }
  group_pointers(e, "  ");
  for (size_t gi = 0; gi < g.groups.size(); ++gi) {
    const AccessGroup& ag = g.groups[gi];
    e.o << "  const GM " << cty(ag.dtype) << "* const p" << gi << " = q" << gi;
    for (int k = 0; k < cd; ++k) if (!ag.structural_zero[k]) e.o << " + i" << k << " * " << e.coef((int)gi, k);
    e.o << ";\n";
  }
  if (RPT > 1) e.o << "//@@SPLIT\n";  // up to here: from the row number to the row's pointers
  // kept per-element values live in registers across stages
  for (size_t i = 0; i < g.prog.size(); ++i)
    if (keep[i] && !g.prog[i].uniform) e.o << "  " << cty(g.prog[i].dtype) << " k" << i << "[" << NP << "][4];\n";
  for (int ph = 0; ph < nph; ++ph) e.o << "  " << cty(g.phases[ph].out_dtype) << " red" << ph << ";\n";

  auto shift_expr = [&](const Instr& in) {
    const AccessGroup& ag = g.groups[in.group];
    std::ostringstream s;
    bool any = false;
    for (int k = 0; k < cd; ++k) {
      if (in.delta[k] == 0 || ag.structural_zero[k]) continue;
      s << (any ? " + " : "") << in.delta[k] << " * " << e.coef(in.group, k);
      any = true;
    }
    if (!any) s << "0";
    return s.str();
  };
  auto name = [&](int i, bool in_loop) -> std::string {
    const Instr& in = g.prog[i];
    if (in.uniform) return "u" + std::to_string(i);
    if (keep[i]) return "k" + std::to_string(i) + "[p][j]";
    (void)in_loop;
    return "t" + std::to_string(i);
  };
  auto expr = [&](int i) -> std::string {
    const Instr& in = g.prog[i];
    switch (in.kind) {
      case IKind::CONST: return e.cst(in.cslot);
      case IKind::UNARY: return Em::unop(in.op, in.dtype, name(in.a, true));
      case IKind::BINARY:
        if (in.op == GR_DIV && in.dtype == GR_F32 && in.b >= 0 && g.prog[in.b].kind == IKind::CONST) return "gr_divc(" + name(in.a, true) + ", " + name(in.b, true) + ")";
        return Em::binop(in.op, in.dtype, name(in.a, true), name(in.b, true));
      case IKind::RED: return "red" + std::to_string(in.phase);
      default: return "0";
    }
  };

  for (int s = 0; s < nstage; ++s) {
    const bool final_stage = s == nph;
    if (final_stage && g.results.empty()) break;
    e.o << "  // ---- " << (final_stage ? "final map" : "reduction phase") << " " << s << "\n";
    // row-uniform values first
    for (int i : stage_instrs[s]) {
      const Instr& in = g.prog[i];
      if (!in.uniform) continue;
      e.o << "  const " << cty(in.dtype) << " u" << i << " = ";
      if (in.kind == IKind::LOAD) e.o << "p" << in.group << "[" << shift_expr(in) << "]";
      else e.o << expr(i);
      e.o << ";\n";
    }
    if (final_stage && g.out_per_row) {
      if (RPT > 1) e.o << "  GR_ROW_RESULT(" << name(g.results[0], false) << ");\n";
      else e.o << "  if (lane == 0 && row_ok) ((GM " << cty(g.out_dtype) << "*)" << e.slot(e.L.out) << ")[row] = " << name(g.results[0], false) << ";\n";
      break;
    }
    const Phase* ph = final_stage ? nullptr : &g.phases[s];
    if (ph) e.o << "  " << cty(ph->out_dtype) << " acc" << s << " = " << Em::identity(*ph) << ";\n";
    if (final_stage)
      e.o << "  GM " << cty(g.out_dtype) << "* const po = (GM " << cty(g.out_dtype) << "*)" << e.slot(e.L.out) << " + row * C;\n";
    bool any_elem = false;
    for (int i : stage_instrs[s]) if (!g.prog[i].uniform) any_elem = true;
    int want = ph ? ph->value : g.results[0];
    if (!any_elem && !(keep[want] && !g.prog[want].uniform) && g.prog[want].uniform) {
      // the combined value does not depend on the column: combine it C times
      // (only sums and extrema exist: a sum of C equal values, an extremum of them)
      // handled below by the generic loop with the uniform name.
    }
    // Long rows: stages whose loads would pile up in registers (values that pass through heavy operations, or that no later
    // stage needs) or that make values to keep by heavy operations, and the positions that may be in flight there.  Where all
    // loaded values are kept anyway, loads that wait for each other cost more (softmax of 1245 x 26936 53.9 us, 58.5 in groups
    // of four positions).
    int n_loads = 0;
    bool heavy = false, passing = false;
    for (int i : stage_instrs[s]) {
      const Instr& in = g.prog[i];
      if (in.uniform) continue;
      if (in.kind == IKind::LOAD) { ++n_loads; passing = passing || !keep[i]; }
      else if (heavy_op(in)) heavy = true;
    }
    const bool in_groups = RT == 1024 && (n_loads ? heavy || passing : heavy && !final_stage);
    const int LONG_POS = n_loads == 1 ? 4 : (n_loads == 2 ? 2 : 1);
    // two bodies: unguarded positions 0..NP-2, guarded last position
    for (int pass = 0; pass < 2; ++pass) {
      const bool guarded = pass == 1;
      if (exact && guarded) continue;
      const int np_unguarded = exact ? NP : NP - 1;
      if (!guarded && np_unguarded == 0) continue;
      if (!guarded) e.o << "#pragma unroll\n  for (int p = 0; p < " << np_unguarded << "; ++p) {\n";
      else e.o << "  { const int p = " << NP - 1 << ";\n";
      e.o << "    const long long c = (long long)p * " << RT * 4 << " + lane * 4;\n";
      // loads of this stage
      for (int i : stage_instrs[s]) {
        const Instr& in = g.prog[i];
        if (in.kind != IKind::LOAD || in.uniform) continue;
        const AccessGroup& ag = g.groups[in.group];
        char cc = access_class(ag, cd);
        std::string base = "p" + std::to_string(in.group) + " + (" + shift_expr(in) + ")";
        e.o << "    " << cty(in.dtype) << " l" << i << "[4];\n";
        std::string idx = cc == '1' ? "(c + " + std::to_string(in.delta[cd]) + ")" : "(c + " + std::to_string(in.delta[cd]) + ") * " + e.coef(in.group, cd);
        std::string step = cc == '1' ? "1" : e.coef(in.group, cd);
        if (cc == '1') {
          if (guarded) e.o << "    if (c + 4 <= C) ";
          else e.o << "    ";
          e.o << "{ const " << vty4(in.dtype) << " w = " << e.ld(in.group, vty4(in.dtype), base + " + " + idx) << "; l" << i << "[0] = w[0]; l" << i
              << "[1] = w[1]; l" << i << "[2] = w[2]; l" << i << "[3] = w[3]; }\n";
          if (guarded)
            e.o << "    else { for (int j = 0; j < 4; ++j) l" << i << "[j] = (c + j < C) ? (" << base << ")[" << idx << " + j] : " << Em::zero(in.dtype) << "; }\n";
        } else {
          e.o << "    for (int j = 0; j < 4; ++j) l" << i << "[j] = " << (guarded ? "(c + j < C) ? " : "") << "(" << base << ")[" << idx << " + j * " << step << "]"
              << (guarded ? " : " + Em::zero(in.dtype) : std::string()) << ";\n";
        }
      }
      if (final_stage && g.out_dtype != GR_I64) e.o << "    " << (g.out_dtype == GR_F32 ? "f4u" : "i4u") << " ov;\n";
      if (ph && RT == 1024) e.o << "    " << cty(ph->out_dtype) << " c4[4];\n";
      e.o << "#pragma unroll\n    for (int j = 0; j < 4; ++j) {\n";
      for (int i : stage_instrs[s]) {
        const Instr& in = g.prog[i];
        if (in.uniform) continue;
        std::string rhs = in.kind == IKind::LOAD ? "l" + std::to_string(i) + "[j]" : expr(i);
        if (keep[i]) e.o << "      k" << i << "[p][j] = " << rhs << ";\n";
        else e.o << "      const " << cty(in.dtype) << " t" << i << " = " << rhs << ";\n";
      }
      if (ph) {
        // (long rows: the elements of a position in pairs first, which shortens the chain of additions to a quarter)
        std::string upd = RT == 1024 ? "c4[j] = " + name(want, true) + ";" : "acc" + std::to_string(s) + " = " + Em::accumulate(g, s, "acc" + std::to_string(s), [&](int i) { return name(i, true); }) + ";";
        if (guarded && RT == 1024) e.o << "      c4[j] = " << Em::identity(*ph) << ";\n";
        if (guarded) e.o << "      if (c + j < C) " << upd << "\n";
        else e.o << "      " << upd << "\n";
      } else {
        if (g.out_dtype == GR_I64) e.o << "      if (row_ok" << (guarded ? " && c + j < C" : "") << ") po[c + j] = " << name(want, true) << ";\n";
        else e.o << "      ov[j] = " << name(want, true) << ";\n";
      }
      e.o << "    }\n";
      if (ph && RT == 1024) {
        const std::string c = "gr_comb" + std::to_string(s);
        e.o << "    acc" << s << " = " << c << "(acc" << s << ", " << c << "(" << c << "(c4[0], c4[1]), " << c << "(c4[2], c4[3])));\n";
      }
      if (final_stage && g.out_dtype != GR_I64) {
        const char* vt = g.out_dtype == GR_F32 ? "f4u" : "i4u";
        const std::string st = (g.nt & 8) ? "__builtin_nontemporal_store(ov, (GM " + std::string(vt) + "*)(po + c))" : "*(GM " + std::string(vt) + "*)(po + c) = ov";
        if (guarded) e.o << "    if (row_ok) { if (c + 4 <= C) " << st << "; else { for (int j = 0; j < 4; ++j) if (c + j < C) po[c + j] = ov[j]; } }\n";
        else e.o << "    if (row_ok) " << st << ";\n";
      }
      // (long rows: an empty statement that the accumulator passes through holds the loads and the temporaries of a few positions
      // at a time in registers; the compiler would sink the arithmetic of all positions behind all loads)
      if (in_groups && !guarded) e.o << "    if (" << (heavy ? "" : "p < " + std::to_string(NP - 2) + " && ") << "p % " << LONG_POS << " == " << LONG_POS - 1 << ") asm volatile(\"\" : " << (ph ? "\"+v\"(acc" + std::to_string(s) + ")" : std::string()) << " : : \"memory\");\n";
      e.o << "  }\n";
    }
    if (ph) {
      e.o << "  acc" << s << " = gr_lanes" << s << "(acc" << s << ");\n";
      if (RT > 64) {
        const char* T = cty(ph->out_dtype);
        e.o << "  { " << T << "* sm = (" << T << "*)gr_sm[" << s << "];\n"
               "    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = acc" << s << ";\n"
               "    __syncthreads();\n";
        if (RT == 1024) {
          e.o << "    " << T << " w[16];\n    for (int q = 0; q < 16; ++q) w[q] = sm[q];\n"
                 "    for (int d = 1; d < 16; d *= 2) for (int q = 0; q < 16; q += 2 * d) w[q] = gr_comb" << s << "(w[q], w[q + d]);\n    acc" << s << " = w[0]; }\n";
        } else if (RT == 256) e.o << "    acc" << s << " = gr_comb" << s << "(gr_comb" << s << "(sm[0], sm[1]), gr_comb" << s << "(sm[2], sm[3])); }\n";
        else e.o << "    const int w0 = (threadIdx.x >> 7) * 2;\n    acc" << s << " = gr_comb" << s << "(sm[w0], sm[w0 + 1]); }\n";
      }
      e.o << "  red" << s << " = acc" << s << ";\n";
    }
  }
  };  // emit_body
  if (RPT == 1) emit_body(false);
  else {
    // the per-row code as text: without column guards for the workgroups whose rows all exist when
    // the rows are exactly as wide as the lanes' positions, with guards for everything else
    std::string body_exact, body_guarded;
    for (int v = 0; v < 2; ++v) {
      std::ostringstream tmp;
      e.o.swap(tmp);
      emit_body(v == 0);
      e.o.swap(tmp);
      (v == 0 ? body_exact : body_guarded) = tmp.str();
    }
    const std::string T = cty(g.out_dtype);
    const std::string out = "((GM " + T + "*)" + e.slot(e.L.out) + ")";
    const std::string mark = "//@@SPLIT\n";
    const std::string setup = body_exact.substr(0, body_exact.find(mark)), stages = body_exact.substr(body_exact.find(mark) + mark.size());
    body_guarded.erase(body_guarded.find(mark), mark.size());
    e.o << "  if (((long long)blockIdx.x * " << RPT << " + " << RPT << ") * " << RB << " <= ROWS && C == " << RT * 4 * NP << ") {\n"
           "    // all rows of the workgroup exist and are exactly as wide as the lanes' positions: no guards;\n"
           "    // the rows' pointers first (index arithmetic with branches), then straight-line code in which\n"
           "    // the loads of the " << RPT << " rows overlap; the results are stored at the end\n"
           "    " << T << " outv[" << RPT << "];\n";
    for (size_t gi = 0; gi < g.groups.size(); ++gi) e.o << "    const GM " << cty(g.groups[gi].dtype) << "* P" << gi << "[" << RPT << "];\n";
    e.o << "#pragma unroll\n    for (int rr = 0; rr < " << RPT << "; ++rr) {\n" << setup;
    for (size_t gi = 0; gi < g.groups.size(); ++gi) e.o << "      P" << gi << "[rr] = p" << gi << ";\n";
    e.o << "    }\n#define GR_ROW_RESULT(v) outv[rr] = (v)\n#pragma unroll\n    for (int rr = 0; rr < " << RPT << "; ++rr) {\n      const bool row_ok = true;\n      (void)row_ok;\n";
    for (size_t gi = 0; gi < g.groups.size(); ++gi) e.o << "      const GM " << cty(g.groups[gi].dtype) << "* const p" << gi << " = P" << gi << "[rr];\n";
    e.o << stages << "    }\n#undef GR_ROW_RESULT\n"
           "    if (lane == 0) {\n";
    for (int rr = 0; rr < RPT; ++rr)
      e.o << "      " << out << "[((long long)blockIdx.x * " << RPT << " + " << rr << ") * " << RB << " + threadIdx.x / " << RT << "] = outv[" << rr << "];\n";
    e.o << "    }\n  } else {\n"
           "#define GR_ROW_RESULT(v) do { if (lane == 0) " << out << "[row] = (v); } while (0)\n"
           "    for (int rr = 0; rr < " << RPT << "; ++rr) {\n      if (((long long)blockIdx.x * " << RPT << " + rr) * " << RB << " + threadIdx.x / " << RT << " >= ROWS) break;\n"
        << body_guarded << "    }\n#undef GR_ROW_RESULT\n  }\n";
  }
  e.o << "}\n";
}

// ---- REDUCE (generic reduction root) --------------------------------------------

void reduce_combine(Em& e, const std::string& squares = "") {
  const GroupPlan& g = e.g;
  const Phase& ph = g.phases[0];
  const char* T = cty(ph.out_dtype);
  // Stage 2 (Section 3.2: "a separate kernel ... only uses the binary operation"): combines the
  // NSPLIT partial results of every output in a fixed order.
  kernel_head(e, kernel_name(g) + "_combine");
  e.o << "  const long long NOUT = " << e.S(e.L.extra) << ", NSPLIT = " << e.S(e.L.extra + 3) << " & 0xffffffffll;\n";
  e.o << "  const GM " << T << "* const ws = (const GM " << T << "*)" << e.slot(e.L.extra + 2) << ";\n";
  e.o << "  GM " << T << "* const out = (GM " << T << "*)" << e.slot(e.L.out) << ";\n";
  const bool moments = !squares.empty();
  if (moments)
    // means and sums of squares about them follow the sums, one per split and output each; the elements per split are known
    e.o << "  const long long LEN = " << e.S(e.L.extra + 1) << ", chunk = (LEN + NSPLIT - 1) / NSPLIT;\n"
           "  const GM float* const wu = ws + NSPLIT * NOUT; const GM float* const wm = wu + NSPLIT * NOUT;\n"
           "  GM float* const sq = (GM float*)" << squares << ";\n"
           "  auto count = [&](long long s) { const long long left = LEN - s * chunk; return (float)(left < 0 ? 0 : (left < chunk ? left : chunk)); };\n";
  // Bound by latency.  Many outputs and many splits: 16 lanes across neighbouring outputs (64 bytes of a split's results) by 16 along
  // the splits, a lane's loads in flight four at a time (a lane per output took all splits in turn, three times over with squares: 25000 x
  // 1024 variances 45.8 -> 28.1 us, sums 24.9 -> 21.3).
  e.o << "  if (NOUT >= 1024 && NSPLIT >= " << kCombineSplits << ") {\n"
         "    const unsigned tx = threadIdx.x % 16, ty = threadIdx.x / 16;\n"
         "    const long long oraw = (long long)blockIdx.x * 16 + tx, o = oraw < NOUT ? oraw : NOUT - 1;\n"
         "    __shared__ " << T << " part[16][17];\n"
         "    auto fold = [&](" << T << " v) {\n      part[ty][tx] = v;\n      __syncthreads();\n      " << T << " w[16];\n"
         "#pragma unroll\n      for (int q = 0; q < 16; ++q) w[q] = part[q][tx];\n"
         "#pragma unroll\n      for (int d = 1; d < 16; d *= 2)\n"
         "#pragma unroll\n        for (int q = 0; q < 16; q += 2 * d) w[q] = gr_comb0(w[q], w[q + d]);\n"
         "      __syncthreads();\n      return w[0];\n    };\n"
         "    " << T << " acc = " << Em::identity(ph) << ";\n";
  if (moments)
    // (a lane's first four splits stay in registers for the second look)
    e.o << "    float u[4], m2[4], t = 0.0f, m = 0.0f;\n"
           "    for (long long s0 = ty; s0 < NSPLIT; s0 += 64) {\n      float x[4], y[4], z[4];\n"
           "#pragma unroll\n      for (int i = 0; i < 4; ++i) { const long long s = s0 + 16 * i, p = s < NSPLIT ? s : s0; x[i] = ws[p * NOUT + o]; y[i] = wu[p * NOUT + o]; z[i] = wm[p * NOUT + o]; }\n"
           "#pragma unroll\n      for (int i = 0; i < 4; ++i) { if (s0 + 16 * i < NSPLIT) { acc += x[i]; t += count(s0 + 16 * i) * y[i]; } if (s0 == ty) { u[i] = y[i]; m2[i] = z[i]; } }\n    }\n"
           "    t = fold(t) / (float)LEN;\n    const float over = gr_overflow(t);\n"
           "    for (long long s0 = ty; s0 < NSPLIT; s0 += 64) {\n      if (s0 != ty) {\n"
           "#pragma unroll\n        for (int i = 0; i < 4; ++i) { const long long s = s0 + 16 * i, p = s < NSPLIT ? s : s0; u[i] = wu[p * NOUT + o]; m2[i] = wm[p * NOUT + o]; }\n      }\n"
           "#pragma unroll\n      for (int i = 0; i < 4; ++i) { const long long s = s0 + 16 * i; const float d = u[i] - t, w = m2[i] + count(s) * d * d; m += s < NSPLIT ? w : 0.0f; }\n    }\n"
           "    m = fold(m) + over;\n";
  else
    e.o << "    for (long long s0 = ty; s0 < NSPLIT; s0 += 64) {\n      " << T << " x[4];\n"
           "#pragma unroll\n      for (int i = 0; i < 4; ++i) { const long long s = s0 + 16 * i; x[i] = ws[(s < NSPLIT ? s : s0) * NOUT + o]; }\n"
           "#pragma unroll\n      for (int i = 0; i < 4; ++i) if (s0 + 16 * i < NSPLIT) acc = gr_comb0(acc, x[i]);\n    }\n";
  e.o << "    acc = fold(acc);\n    if (ty == 0 && oraw < NOUT) {\n" << (moments ? "      sq[o] = gr_squares(acc, m);\n" : "") << "      out[o] = acc;\n    }\n    return;\n  }\n"
         "  __shared__ long long gr_sm[4];\n";
  if (moments)
    e.o << "  if (NOUT >= 1024) {\n"
           "    const long long o = (long long)blockIdx.x * 256 + threadIdx.x;\n    if (o < NOUT) {\n"
           "      float a[8] = {0, 0, 0, 0, 0, 0, 0, 0};\n"
           "      for (long long s = 0; s < NSPLIT; s += 8)\n"
           "#pragma unroll\n        for (int i = 0; i < 8; ++i) { const bool in = s + i < NSPLIT; const long long p = in ? s + i : 0; const float w = count(p) * wu[p * NOUT + o]; a[i] += in ? w : 0.0f; }\n"
           "      float t = (((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]))) / (float)LEN;\n"
           "      const float over = gr_overflow(t);\n"
           "#pragma unroll\n      for (int i = 0; i < 8; ++i) a[i] = 0.0f;\n"
           "      for (long long s = 0; s < NSPLIT; s += 8)\n"
           "#pragma unroll\n        for (int i = 0; i < 8; ++i) { const bool in = s + i < NSPLIT; const long long p = in ? s + i : 0; const float d = wu[p * NOUT + o] - t, w = wm[p * NOUT + o] + count(p) * d * d; a[i] += in ? w : 0.0f; }\n"
           "      sq[o] = (((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]))) + over;\n    }\n  } else {\n"
           // (a lane's first two splits, all of them as a rule, loaded at once and kept for the second look: three round trips to memory
           // of 2 us each were one after the other)
           "    const long long o = blockIdx.x;\n    float* const sm = (float*)gr_sm;\n    float acc = 0.0f, t = 0.0f, m = 0.0f, u[2], m2[2];\n"
           "    for (long long s0 = threadIdx.x; s0 < NSPLIT; s0 += 512) {\n      float x[2], y[2], z[2];\n"
           "#pragma unroll\n      for (int i = 0; i < 2; ++i) { const long long s = s0 + 256 * i, p = s < NSPLIT ? s : s0; x[i] = ws[p * NOUT + o]; y[i] = wu[p * NOUT + o]; z[i] = wm[p * NOUT + o]; }\n"
           "#pragma unroll\n      for (int i = 0; i < 2; ++i) { if (s0 + 256 * i < NSPLIT) { acc += x[i]; t += count(s0 + 256 * i) * y[i]; } if (s0 == threadIdx.x) { u[i] = y[i]; m2[i] = z[i]; } }\n    }\n"
           "    t = gr_lanes0(t);\n    acc = gr_lanes0(acc);\n    if ((threadIdx.x & 63) == 0) { sm[threadIdx.x >> 6] = t; sm[4 + (threadIdx.x >> 6)] = acc; }\n    __syncthreads();\n"
           "    t = ((sm[0] + sm[1]) + (sm[2] + sm[3])) / (float)LEN;\n    acc = (sm[4] + sm[5]) + (sm[6] + sm[7]);\n    __syncthreads();\n    const float over = gr_overflow(t);\n"
           "    for (long long s0 = threadIdx.x; s0 < NSPLIT; s0 += 512) {\n      if (s0 != threadIdx.x) {\n"
           "#pragma unroll\n        for (int i = 0; i < 2; ++i) { const long long s = s0 + 256 * i, p = s < NSPLIT ? s : s0; u[i] = wu[p * NOUT + o]; m2[i] = wm[p * NOUT + o]; }\n      }\n"
           "#pragma unroll\n      for (int i = 0; i < 2; ++i) { const long long s = s0 + 256 * i; const float d = u[i] - t, w = m2[i] + count(s) * d * d; m += s < NSPLIT ? w : 0.0f; }\n    }\n"
           "    m = gr_lanes0(m);\n    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = m;\n    __syncthreads();\n"
           "    if (threadIdx.x == 0) { sq[o] = gr_squares(acc, ((sm[0] + sm[1]) + (sm[2] + sm[3])) + over); out[o] = acc; }\n    return;\n  }\n";
  e.o << "  if (NOUT >= 1024) {\n"
         "    const long long o = (long long)blockIdx.x * 256 + threadIdx.x;\n"
         "    if (o < NOUT) {\n      " << T << " acc = ws[o];\n"
         "      long long s = 1;\n"
         "      for (; s + 8 <= NSPLIT; s += 8) {\n"   // eight independent loads in flight, combined in a fixed order, pairs first
         "        const " << T << " v0 = ws[s * NOUT + o], v1 = ws[(s + 1) * NOUT + o], v2 = ws[(s + 2) * NOUT + o], v3 = ws[(s + 3) * NOUT + o];\n"
         "        const " << T << " v4 = ws[(s + 4) * NOUT + o], v5 = ws[(s + 5) * NOUT + o], v6 = ws[(s + 6) * NOUT + o], v7 = ws[(s + 7) * NOUT + o];\n"
         "        acc = gr_comb0(acc, gr_comb0(gr_comb0(gr_comb0(v0, v1), gr_comb0(v2, v3)), gr_comb0(gr_comb0(v4, v5), gr_comb0(v6, v7))));\n"
         "      }\n"
         "      for (; s < NSPLIT; ++s) acc = gr_comb0(acc, ws[s * NOUT + o]);\n"
      << (squares.empty() ? "" : "      sq[o] = gr_squares(acc, sq[o]);\n")
      << "      out[o] = acc;\n    }\n"
         "    return;\n  }\n";
  if (!moments)
    e.o << "  const long long o = blockIdx.x;\n  " << T << " acc = " << Em::identity(ph) << ";\n"
           "  for (long long s = threadIdx.x; s < NSPLIT; s += 256) acc = gr_comb0(acc, ws[s * NOUT + o]);\n"
           "  acc = gr_lanes0(acc);\n"
           "  " << T << "* sm = (" << T << "*)gr_sm;\n"
           "  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = acc;\n"
           "  __syncthreads();\n"
           "  if (threadIdx.x == 0) out[o] = gr_comb0(gr_comb0(sm[0], sm[1]), gr_comb0(sm[2], sm[3]));\n";
  e.o << "}\n";
}

// One kernel of mode 0 (see gen_reduce_columns).  Loads in flight per lane and array: U, written out, all first (a wave-wide
// vote in the body keeps the compiler from unrolling a loop with a remainder); what is left of a lane's share is loaded together
// with clamped positions, whose surplus values are not combined.
// `squares` (an expression for the output pointer): the sums of squared deviations from the mean come out of the same pass, the sums
// being what they are without.  A lane takes a batch's mean and squares about it and joins them to its running mean and
// squares (n1 n2 / (n1 + n2) times the squared difference of the means is what a join adds), which loses no digits however
// far the mean is from zero, because means are relative to the median of three of the column's values (no outlier) and a
// value is subtracted from once, as in the second of two passes.  Partial results of
// lanes and of splits are joined the same way, all at once about their common mean.
// Means stay finite: values so far apart that a difference of means overflows (or a sum of them below) have infinite squares, and a
// batch that holds a value that is not finite has squares that are not a number; neither enters the mean.
void reduce_columns_kernel(Em& e, bool wide, int U, const std::string& squares = "") {
  const bool moments = !squares.empty();
  const GroupPlan& g = e.g;
  const int rank = g.rank, kr = g.red_kept_rank, kd = kr - 1;
  const Phase& ph = g.phases[0];
  const char* T = cty(ph.out_dtype);
  const int W = g.red_vec ? 4 : 1;
  kernel_head(e, kernel_name(g) + (wide ? "_wide" : ""), kReduceLanes);
  e.o << "  const long long NOUT = " << e.S(e.L.extra) << ", LEN = " << e.S(e.L.extra + 1) << ", NSPLIT = " << e.S(e.L.extra + 3) << " & 0xffffffffll;\n"
         "  const unsigned BX = (unsigned)(" << e.slot(e.L.extra + 3) << " >> 32), BY = " << kReduceLanes << "u / BX;\n"
         "  const unsigned ty = threadIdx.x / BX, tx = threadIdx.x - ty * BX;\n"
         "  const long long D = " << e.dim(kd) << ", VD = (D + " << W - 1 << ") / " << W << ", V = " << (kr == 1 ? "VD" : "NOUT / D * VD") << ";\n"
         "  const long long blocks_o = (V + BX - 1) / BX;\n"
         "  long long orem = (long long)(blockIdx.x % blocks_o) * BX + tx;\n"
         "  const long long split = blockIdx.x / blocks_o;\n"
         "  const bool ok = orem < V && ty < BY;\n"
         "  if (!ok) orem = 0;\n"
         "  const long long chunk = (LEN + NSPLIT - 1) / NSPLIT, jbeg = split * chunk, jend = (jbeg + chunk < LEN) ? jbeg + chunk : LEN;\n";
  if (kr == 1) e.o << "  const long long v" << kd << " = orem;\n";
  else e.o << "  const long long v" << kd << " = gr_peel(orem, VD);\n";
  if (W == 4) e.o << "  const long long i" << kd << " = 4 * v" << kd << " + 4 <= D ? 4 * v" << kd << " : D - 4;\n";
  else e.o << "  const long long i" << kd << " = v" << kd << ";\n";
  e.o << "  const long long o = " << (kr == 1 ? "" : "orem * D + ") << "i" << kd << ";\n";
  for (int k = kd - 1; k >= 0; --k) {
    if (k == 0) e.o << "  const long long i0 = orem;\n";
    else e.o << "  const long long i" << k << " = gr_peel(orem, " << e.dim(k) << ");\n";
  }
  group_pointers(e, "  ");
  for (size_t gi = 0; gi < g.groups.size(); ++gi) {
    const AccessGroup& ag = g.groups[gi];
    e.o << "  const GM " << cty(ag.dtype) << "* const p" << gi << " = q" << gi;
    for (int k = 0; k < kr; ++k) if (!ag.structural_zero[k]) e.o << " + i" << k << " * " << e.coef((int)gi, k);
    e.o << ";\n";
  }
  for (int c = 0; c < W; ++c) e.o << "  " << T << " acc" << c << " = " << Em::identity(ph) << ";\n";
  if (moments) {
    e.o << "  float count = 0.0f;\n";
    for (int c = 0; c < W; ++c) e.o << "  float mu" << c << " = 0.0f, m2" << c << " = 0.0f, pv" << c << " = 0.0f;\n";
  }
  auto loads = [&](int u, const std::string& jx, const char* ind) {
    const std::string su = "_" + std::to_string(u);
    if (rank > kr) {
      e.o << ind << "long long jrem" << su << " = " << jx << ";\n";
      for (int k = rank - 1; k >= kr; --k) {
        if (k == kr) e.o << ind << "const long long i" << k << su << " = jrem" << su << ";\n";
        else e.o << ind << "const long long i" << k << su << " = gr_peel(jrem" << su << ", " << e.dim(k) << ");\n";
      }
    }
    for (size_t i = 0; i < g.prog.size(); ++i) {
      const Instr& in = g.prog[i];
      if (in.kind != IKind::LOAD) continue;
      const AccessGroup& ag = g.groups[in.group];
      std::ostringstream at;
      at << "p" << in.group << " + 0";
      for (int k = 0; k < rank; ++k) {
        if (ag.structural_zero[k]) continue;
        if (k >= kr) at << " + (i" << k << su << " + " << in.delta[k] << ") * " << e.coef(in.group, k);
        else if (in.delta[k]) at << " + " << in.delta[k] << " * " << e.coef(in.group, k);
      }
      if (W == 1 || ag.structural_zero[kd]) e.o << ind << "const " << cty(in.dtype) << " w" << i << su << " = (" << at.str() << ")[0];\n";
      else e.o << ind << "const " << vty4(in.dtype) << " w" << i << su << " = " << e.ld(in.group, vty4(in.dtype), at.str()) << ";\n";
    }
  };
  // values of element u: v<u>_<c>
  auto values = [&](int u) {
    const std::string su = "_" + std::to_string(u);
    for (int c = 0; c < W; ++c) {
      const std::string pre = "t" + std::to_string(c) + "_";
      e.o << "      " << T << " v" << u << "_" << c << ";\n      {\n";
      emit_scalar_program(e, g.prog, {ph.value},
                          [&](const Instr& in, int id) {
                            const std::string w = "w" + std::to_string(id) + su;
                            return W == 1 || g.groups[in.group].structural_zero[kd] ? w : w + "[" + std::to_string(c) + "]";
                          },
                          "0.0f", pre, "        ");
      e.o << "        v" << u << "_" << c << " = " << pre << ph.value << ";\n      }\n";
    }
  };
  auto join = [&](const char* to, int u) {
    for (int c = 0; c < W; ++c) e.o << "      " << to << c << " = gr_comb0(" << to << c << ", v" << u << "_" << c << ");\n";
  };
  // A chain of additions as long as a lane's share of the range loses digits (4096 x 262144 uniform values, relative error 2.2e-7
  // with one, 1.2e-7 with chunks of 512): the wide kernel adds up 64 elements before they join the accumulator.  The other
  // one's shares are short (choose_column_split); its registers are worth more.
  const std::string more = "j + " + std::to_string(U - 1) + "ll * BY < jend";
  const bool blocked = wide && ph.op == GR_SUM && ph.out_dtype == GR_F32;
  const char* const to = blocked ? "b" : "acc";
  e.o << "  if (ok) {\n    long long j = jbeg + ty;\n";
  if (moments) {
    e.o << "    {\n";
    loads(U, "0ll", "      ");
    loads(U + 1, "LEN / 2", "      ");
    loads(U + 2, "LEN - 1", "      ");
    for (int u = U; u < U + 3; ++u) values(u);
    for (int c = 0; c < W; ++c) {
      e.o << "      pv" << c << " = __builtin_amdgcn_fmed3f(";
      for (int u = U; u < U + 3; ++u) e.o << "v" << u << "_" << c << (u < U + 2 ? ", " : ");\n");
    }
    e.o << "    }\n";
  }
  if (blocked) {
    e.o << "    while (" << more << ") {\n";
    for (int c = 0; c < W; ++c) e.o << "      " << T << " b" << c << " = " << Em::identity(ph) << ";\n";
  }
  e.o << "    for (" << (blocked ? "int n = 0; n < " + std::to_string(64 / U) + " && " : std::string("; ")) << more << "; " << (blocked ? "++n, " : "") << "j += " << U << "ll * BY) {\n";
  for (int u = 0; u < U; ++u) loads(u, "j + " + std::to_string(u) + "ll * BY", "      ");
  e.o << "      __builtin_amdgcn_sched_barrier(0);\n";
  if (blocked) {   // (pairs first)
    std::function<void(int, int)> tree = [&](int lo, int n) {
      if (n == 1) { values(lo); return; }
      tree(lo, n / 2);
      tree(lo + n / 2, n / 2);
      join(("v" + std::to_string(lo) + "_").c_str(), lo + n / 2);
    };
    tree(0, U);
    join(to, 0);
  } else if (moments) {
    for (int u = 0; u < U; ++u) { values(u); join(to, u); }
    e.o << "      count += " << U << ".0f;\n      const float share = " << U << ".0f / count, rest = count - " << U << ".0f;\n";
    auto v = [](int u, int c) { return "v" + std::to_string(u) + "_" + std::to_string(c); };
    std::function<std::string(int, int, int, bool)> sum = [&](int c, int lo, int n, bool rel) {
      if (n == 1) return rel ? "(" + v(lo, c) + " - pv" + std::to_string(c) + ")" : v(lo, c);
      return "(" + sum(c, lo, n / 2, rel) + " + " + sum(c, lo + n / 2, n - n / 2, rel) + ")";
    };
    auto join_batch = [&](int c) {
      const std::string C = std::to_string(c);
      e.o << "        { const float at = pv" << C << " + m" << C << ";\n";
      for (int u = 0; u < U; ++u) e.o << "        " << v(u, c) << " -= at; " << v(u, c) << " *= " << v(u, c) << ";\n";
      e.o << "        mu" << C << " = __builtin_fmaf(d" << C << ", share, mu" << C << "); m2" << C << " += " << sum(c, 0, U, false) << " + d" << C << " * (rest * share) * d" << C << "; }\n";
    };
    for (int c = 0; c < W; ++c) e.o << "      const float m" << c << " = " << sum(c, 0, U, true) << " * " << std::to_string(1.0 / U) << "f, d" << c << " = m" << c << " - mu" << c << ";\n";
    e.o << "      if (";
    for (int c = 0; c < W; ++c) e.o << (c ? " & " : "") << "(__builtin_fabsf(d" << c << ") < __builtin_inff())";
    e.o << ") {\n";   // (one branch for all columns: the compiler interleaves their arithmetic)
    for (int c = 0; c < W; ++c) join_batch(c);
    e.o << "      } else {\n";
    for (int c = 0; c < W; ++c) {
      e.o << "        if (__builtin_fabsf(d" << c << ") < __builtin_inff())\n";
      join_batch(c);
      e.o << "        else m2" << c << " += ";
      for (int u = 0; u < U; ++u) e.o << (u ? " && " : "") << "__builtin_fabsf(" << v(u, c) << ") < __builtin_inff()";
      e.o << " ? __builtin_inff() : __builtin_nanf(\"\");\n";
    }
    e.o << "      }\n";
  } else
    for (int u = 0; u < U; ++u) { e.o << "      {\n"; values(u); join(to, u); e.o << "      }\n"; }
  e.o << "    }\n";
  if (blocked) {
    for (int c = 0; c < W; ++c) e.o << "    acc" << c << " = gr_comb0(acc" << c << ", b" << c << ");\n";
    e.o << "    }\n";
  }
  if (U > 1) {
    e.o << "    if (j < jend) {\n";
    for (int u = 0; u + 1 < U; ++u) loads(u, u == 0 ? std::string("j") : "(j + " + std::to_string(u) + "ll * BY < jend ? j + " + std::to_string(u) + "ll * BY : j)", "      ");
    e.o << "      __builtin_amdgcn_sched_barrier(0);\n";
    for (int u = 0; u + 1 < U; ++u) {
      e.o << "      " << (u ? "if (j + " + std::to_string(u) + "ll * BY < jend) " : std::string()) << "{\n";
      values(u);
      join("acc", u);
      if (moments) {
        e.o << "      count += 1.0f;\n      const float share = 1.0f / count;\n";
        auto join_one = [&](int c) { e.o << "        { mu" << c << " = __builtin_fmaf(d" << c << ", share, mu" << c << "); m2" << c << " += d" << c << " * ((count - 1.0f) * share) * d" << c << "; }\n"; };
        for (int c = 0; c < W; ++c) e.o << "      const float d" << c << " = v" << u << "_" << c << " - pv" << c << " - mu" << c << ";\n";
        e.o << "      if (";
        for (int c = 0; c < W; ++c) e.o << (c ? " & " : "") << "(__builtin_fabsf(d" << c << ") < __builtin_inff())";
        e.o << ") {\n";
        for (int c = 0; c < W; ++c) join_one(c);
        e.o << "      } else {\n";
        for (int c = 0; c < W; ++c) {
          e.o << "        if (__builtin_fabsf(d" << c << ") < __builtin_inff())\n";
          join_one(c);
          e.o << "        else m2" << c << " += __builtin_fabsf(v" << u << "_" << c << ") < __builtin_inff() ? __builtin_inff() : __builtin_nanf(\"\");\n";
        }
        e.o << "      }\n";
      }
      e.o << "      }\n";
    }
    e.o << "    }\n";
  }
  e.o << "  }\n";
  e.o << "  GM " << T << "* const dst = NSPLIT > 1 ? (GM " << T << "*)" << e.slot(e.L.extra + 2) << " + split * NOUT : (GM " << T << "*)" << e.slot(e.L.out) << ";\n";
  if (moments) {
    // the lanes of an output: their common mean, then their squares and those of their means about it
    e.o << "  GM float* const wsu = (GM float*)" << e.slot(e.L.extra + 2) << " + (NSPLIT + split) * NOUT;\n"
           "  GM float* const dst2 = NSPLIT > 1 ? wsu + NSPLIT * NOUT : (GM float*)" << squares << ";\n"
           "  {\n    __shared__ float sn[" << kReduceLanes << "], su[" << W << "][" << kReduceLanes << "], sq[" << W << "][" << kReduceLanes << "];\n"
           "    sn[threadIdx.x] = ok ? count : 0.0f;\n";
    for (int c = 0; c < W; ++c) e.o << "    su[" << c << "][threadIdx.x] = mu" << c << "; sq[" << c << "][threadIdx.x] = m2" << c << ";\n";
    e.o << "    __syncthreads();\n"
           "    auto meet = [&](int c, unsigned first, unsigned step, unsigned end, float& n, float& u, float& m) {\n"
           "      n = 0.0f;\n      float a[8] = {0, 0, 0, 0, 0, 0, 0, 0};\n"   // (eight chains: no long one)
           "      for (unsigned q = first; q < end; q += 8 * step)\n"
           "#pragma unroll\n        for (int i = 0; i < 8; ++i) { const bool in = q + i * step < end; const unsigned at = (in ? q + i * step : first) * BX + tx; const float k = in ? sn[at] : 0.0f, w = su[c][at]; n += k; a[i] += in ? k * w : 0.0f; }\n"
           "      u = n > 0.0f ? (((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]))) / n : 0.0f;\n      const float over = gr_overflow(u);\n"
           "#pragma unroll\n      for (int i = 0; i < 8; ++i) a[i] = 0.0f;\n"
           "      for (unsigned q = first; q < end; q += 8 * step)\n"
           "#pragma unroll\n        for (int i = 0; i < 8; ++i) { const bool in = q + i * step < end; const unsigned at = (in ? q + i * step : first) * BX + tx; const float d = su[c][at] - u, w = sq[c][at] + sn[at] * d * d; a[i] += in ? w : 0.0f; }\n"
           "      m = (((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]))) + over;\n    };\n"
           // (lanes past the rows of a short range have nothing; many lanes meet in groups first, a lane per group and column)
           "    const unsigned have = jend - jbeg < BY ? (unsigned)(jend > jbeg ? jend - jbeg : 0) : BY;\n"
           "    unsigned nl = have;\n"
           "    if (have > 16) {\n      const unsigned G = have >= 64 ? 16 : have / 4, c = ty % 4, g = ty / 4;\n      float n = 0.0f, u = 0.0f, m = 0.0f;\n"
           "      const bool here = ok && g < G && c < " << W << "u;\n      if (here) meet((int)c, g, G, have, n, u, m);\n"
           "      __syncthreads();\n"
           "      if (here) { if (c == 0) sn[g * BX + tx] = n; su[c][g * BX + tx] = u; sq[c][g * BX + tx] = m; }\n"
           "      __syncthreads();\n      nl = G;\n    }\n"
           "    if (ok) for (unsigned c = ty; c < " << W << "u; c += BY) {\n      float n, u, m;\n      meet((int)c, 0, 1, nl, n, u, m);\n      if (NSPLIT > 1) wsu[o + c] = u;\n      dst2[o + c] = m;\n    }\n  }\n";
  }
  e.o << "  if (BY == 1) {\n    if (ok) { ";
  for (int c = 0; c < W; ++c) e.o << "dst[o + " << c << "] = acc" << c << "; " << (moments ? "if (NSPLIT == 1) dst2[o + " + std::to_string(c) + "] = gr_squares(acc" + std::to_string(c) + ", dst2[o + " + std::to_string(c) + "]); " : "");
  e.o << "}\n    return;\n  }\n"
         "  __shared__ " << T << " sm[" << W << "][" << kReduceLanes << "];\n";
  for (int c = 0; c < W; ++c) e.o << "  sm[" << c << "][threadIdx.x] = acc" << c << ";\n";
  // (many lanes to an output: sixteen of them first, in four chains where they are very many, so that no lane adds many partial results in turn)
  e.o << "  __syncthreads();\n  unsigned ny = BY;\n  if (BY > 16) {\n    if (ok && ty < 16) {\n      unsigned q = ty + 16;\n      if (BY >= 128) {\n";
  for (int c = 0; c < W; ++c) e.o << "        " << T << " f" << c << "_0 = acc" << c << ", f" << c << "_1 = " << Em::identity(ph) << ", f" << c << "_2 = f" << c << "_1, f" << c << "_3 = f" << c << "_1;\n";
  e.o << "        for (; q + 48 < BY; q += 64) {\n";
  for (int c = 0; c < W; ++c)
    for (int u = 0; u < 4; ++u) e.o << "          f" << c << "_" << u << " = gr_comb0(f" << c << "_" << u << ", sm[" << c << "][(q + " << 16 * u << ") * BX + tx]);\n";
  e.o << "        }\n";
  for (int c = 0; c < W; ++c) e.o << "        acc" << c << " = gr_comb0(gr_comb0(f" << c << "_0, f" << c << "_1), gr_comb0(f" << c << "_2, f" << c << "_3));\n";
  e.o << "      }\n      for (; q < BY; q += 16) {\n";
  for (int c = 0; c < W; ++c) e.o << "        acc" << c << " = gr_comb0(acc" << c << ", sm[" << c << "][q * BX + tx]);\n";
  e.o << "      }\n";
  e.o << "    }\n    __syncthreads();\n    if (ok && ty < 16) {\n";
  for (int c = 0; c < W; ++c) e.o << "      sm[" << c << "][threadIdx.x] = acc" << c << ";\n";
  e.o << "    }\n    __syncthreads();\n    ny = 16;\n  }\n"
         "  if (ok) for (unsigned c = ty; c < " << W << "u; c += BY) {\n"
         "    " << T << " r = sm[c][tx];\n"
         "    unsigned q = 1;\n"
         "    for (; q + 8 <= ny; q += 8) {\n"   // eight LDS reads in flight, pairs first
         "      " << T << " w[8];\n"
         "#pragma unroll\n      for (int u = 0; u < 8; ++u) w[u] = sm[c][(q + u) * BX + tx];\n"
         "      r = gr_comb0(r, gr_comb0(gr_comb0(gr_comb0(w[0], w[1]), gr_comb0(w[2], w[3])), gr_comb0(gr_comb0(w[4], w[5]), gr_comb0(w[6], w[7]))));\n"
         "    }\n"
         "    " << T << " rest = " << Em::identity(ph) << ";\n"
         "    for (; q < ny; ++q) rest = gr_comb0(rest, sm[c][q * BX + tx]);\n"
         "    r = gr_comb0(r, rest);\n"
         "    dst[o + c] = r;\n"
      << (moments ? "    if (NSPLIT == 1) dst2[o + c] = gr_squares(r, dst2[o + c]);\n" : "") << "  }\n}\n";
}

// Mode 0: the kept dimension is the contiguous one (column sums).  A workgroup of 512 lanes is BX
// lanes across the outputs by BY = 512 / BX along the reduced range; a lane takes four consecutive
// outputs with one dwordx4 per array and reduced element (one output where the kept dimension is
// strided or shorter than four) and every BY-th element of its chunk, the BY partial results of an
// output are combined in order through LDS.  BX is an argument: the planner fits it to the shape.
// The last group of four outputs of a ragged dimension starts four from its end: it overlaps the
// group before it, both store the same values, and no load leaves the array.
void gen_reduce_columns(Em& e, const std::string& squares) {
  const GroupPlan& g = e.g;
  const int rank = g.rank, kr = g.red_kept_rank, kd = kr - 1;
  const Phase& ph = g.phases[0];
  const char* T = cty(ph.out_dtype);
  const int W = g.red_vec ? 4 : 1;
  int n_loads = 0;
  for (const Instr& in : g.prog) if (in.kind == IKind::LOAD) ++n_loads;
  // Two kernels, one per kind of shape.  Outputs that fill the chip by themselves (red_wide): batches of four; their workgroups walk
  // rows far apart, and more rows at a time cost more than the loads in flight gain (512 x 2^19: 172.8 us with eight,
  // 166.3 with four; 2048 x 65536 products of two arrays 218 / 176).  Others: batches of eight (16384 x 4096 56.1 us with four, 50.1),
  // whose registers would halve the wavefronts of the former (3 x 2^22 14.7 us from one kernel with both, 13.3).
  // (registers for what a batch loads, of the 256 that 512 lanes leave each: 223 for five arrays by four, 204 for eight by two;
  // twelve by four spilled 1 KiB per lane)
  // Squares about a mean as the second of two passes gives them: about a mean that is not a number, not a number; about an infinite
  // one (the sum overflows, or a value is infinite), infinite for finite values.  gr_overflow: what a mean of means adds to
  // the squares, and zero in its place where it overflows, which only values with infinite squares can make it do.
  if (!squares.empty())
    e.o << "static __device__ __forceinline__ float gr_squares(float s, float m) { return __builtin_fabsf(s) < __builtin_inff() ? m : (s != s ? s : (m == m ? __builtin_inff() : m)); }\n"
           "static __device__ __forceinline__ float gr_overflow(float& mean) { if (__builtin_fabsf(mean) < __builtin_inff()) return 0.0f; mean = 0.0f; return __builtin_inff(); }\n";
  const int most = n_loads <= 5 ? 4 : (n_loads <= 8 ? 2 : 1);
  reduce_columns_kernel(e, false, n_loads <= 2 && g.prog.size() <= 12 ? 8 : most, squares);
  if (squares.empty()) reduce_columns_kernel(e, true, most);
  reduce_combine(e, squares);
}

void gen_reduce(Em& e, const std::string& squares = "") {
  const GroupPlan& g = e.g;
  const int rank = g.rank, kr = g.red_kept_rank;
  const Phase& ph = g.phases[0];
  const char* T = cty(ph.out_dtype);
  prelude(e);
  phase_helpers(e, 0, 64);
  // Stage 1 (Section 3.2: map fused with a per-block combine): every output's reduced range is
  // cut into NSPLIT chunks; a column of lanes (mode 0) or a workgroup (mode 1) combines one chunk.
  if (g.red_mode == 0) { gen_reduce_columns(e, squares); return; }
  kernel_head(e, kernel_name(g));
  e.o << "  const long long NOUT = " << e.S(e.L.extra) << ", LEN = " << e.S(e.L.extra + 1) << ", NSPLIT = " << e.S(e.L.extra + 3) << ";\n";
  e.o << "  const long long o = blockIdx.x % NOUT, split = blockIdx.x / NOUT;\n  __shared__ long long gr_sm[4];\n";
  e.o << "  const long long chunk = (LEN + NSPLIT - 1) / NSPLIT, jbeg = split * chunk, jend = (jbeg + chunk < LEN) ? jbeg + chunk : LEN;\n";
  e.o << "  long long orem = o;\n";
  for (int k = kr - 1; k >= 0; --k) {
    if (k == 0) e.o << "  const long long i0 = orem;\n";
    else e.o << "  const long long i" << k << " = gr_peel(orem, " << e.dim(k) << ");\n";
  }
  group_pointers(e, "  ");
  for (size_t gi = 0; gi < g.groups.size(); ++gi) {
    const AccessGroup& ag = g.groups[gi];
    e.o << "  const GM " << cty(ag.dtype) << "* const p" << gi << " = q" << gi;
    for (int k = 0; k < kr; ++k) if (!ag.structural_zero[k]) e.o << " + i" << k << " * " << e.coef((int)gi, k);
    e.o << ";\n";
  }
  e.o << "  " << T << " acc = " << Em::identity(ph) << ";\n";
  // mode 1 over one contiguous reduced dimension: lanes take four consecutive elements with one
  // dwordx4 per array and keep four partial results; the ragged end goes through the scalar loop
  // (several reduced dimensions: the same when the innermost one holds a multiple of four, so that
  // four consecutive elements never straddle it; chunks are then cut at multiples of four)
  const int rd = rank - 1;
  bool vec = g.red_mode == 1 && rank > kr && (rank == kr + 1 || g.red_vec);
  for (size_t i = 0; vec && i < g.prog.size(); ++i) {
    const Instr& in = g.prog[i];
    if (in.dtype == GR_I64) vec = false;
    if (in.kind == IKind::LOAD && !g.groups[in.group].structural_zero[rd] && access_class(g.groups[in.group], rd) != '1') vec = false;
  }
  if (vec && rank > kr + 1) e.o << "  const long long chunk4 = (chunk + 3) / 4 * 4, jbeg4 = split * chunk4, jend4 = (jbeg4 + chunk4 < LEN) ? jbeg4 + chunk4 : LEN;\n";
  if (vec) {
    const bool multi = rank > kr + 1;
    const char* jb = multi ? "jbeg4" : "jbeg";
    const char* je = multi ? "jend4" : "jend";
    e.o << "  long long j = " << jb << " + 4 * (long long)threadIdx.x;\n  {\n    " << T << " acc1 = acc, acc2 = acc, acc3 = acc;\n";
    // Four vector loads per array in flight: the loop body is written out four times here, all loads first, because the
    // compiler cannot unroll a loop with a remainder once the body holds a wave-wide vote (the math helpers' tests for
    // rare arguments), and one load in flight per lane leaves HBM waiting (measured on sum(sqrt(x)) over 2^27 elements).
    // Every accumulator still takes its elements in increasing order of j: the same sums as a loop of single steps.
    const int U = 4;
    auto emit_loads = [&](int u, const char* ind) {
      const std::string su = "_" + std::to_string(u), jx = "(j + " + std::to_string(1024 * u) + ")";
      if (multi) {
        e.o << ind << "long long jrem" << su << " = " << jx << ";\n";
        for (int k = rank - 1; k >= kr; --k) {
          if (k == kr) e.o << ind << "const long long i" << k << su << " = jrem" << su << ";\n";
          else e.o << ind << "const long long i" << k << su << " = gr_peel(jrem" << su << ", " << e.dim(k) << ");\n";
        }
      } else e.o << ind << "const long long i" << kr << su << " = " << jx << ";\n";
      for (size_t i = 0; i < g.prog.size(); ++i) {
        const Instr& in = g.prog[i];
        if (in.kind != IKind::LOAD) continue;
        const AccessGroup& ag = g.groups[in.group];
        std::ostringstream base;
        base << "p" << in.group << " + 0";
        for (int k = 0; k < kr; ++k) if (!ag.structural_zero[k] && in.delta[k]) base << " + " << in.delta[k] << " * " << e.coef(in.group, k);
        for (int k = kr; k < rank; ++k) {
          if (ag.structural_zero[k]) continue;
          if (k == rd) base << " + i" << k << su << " + " << in.delta[k];
          else base << " + (i" << k << su << " + " << in.delta[k] << ") * " << e.coef(in.group, k);
        }
        if (ag.structural_zero[rd]) e.o << ind << "const " << cty(in.dtype) << " u" << i << su << " = (" << base.str() << ")[0];\n";
        else e.o << ind << "const " << vty4(in.dtype) << " w" << i << su << " = " << e.ld(in.group, vty4(in.dtype), base.str()) << ";\n";
      }
    };
    auto emit_compute = [&](int u, const std::string& ind) {
      const std::string su = "_" + std::to_string(u);
      e.o << ind << "{\n";
      for (int k = rank - 1; k >= kr; --k) e.o << ind << "  const long long i" << k << " = i" << k << su << "; (void)i" << k << ";\n";
      for (int c4 = 0; c4 < 4; ++c4) {
        const std::string pre = "v" + std::to_string(c4) + "_";
        emit_scalar_program(e, g.prog, {ph.value},
                            [&](const Instr& in, int id) {
                              const AccessGroup& ag = g.groups[in.group];
                              if (ag.structural_zero[rd]) return "u" + std::to_string(id) + su;
                              return "w" + std::to_string(id) + su + "[" + std::to_string(c4) + "]";
                            },
                            "0.0f", pre, (ind + "  ").c_str());
        const std::string a = c4 == 0 ? "acc" : "acc" + std::to_string(c4);
        e.o << ind << "  " << a << " = " << Em::combine(ph, a, pre + std::to_string(ph.value)) << ";\n";
      }
      e.o << ind << "}\n";
    };
    e.o << "    for (; j + " << 4 + 1024 * (U - 1) << " <= " << je << "; j += " << 1024 * U << ") {\n";
    for (int u = 0; u < U; ++u) emit_loads(u, "      ");
    e.o << "      __builtin_amdgcn_sched_barrier(0);\n";   // (or the scheduler waits for the first load before it issues the others)
    for (int u = 0; u < U; ++u) emit_compute(u, "      ");
    e.o << "    }\n";
    e.o << "    for (; j + 4 <= " << je << "; j += 1024) {\n";
    emit_loads(0, "      ");
    emit_compute(0, "      ");
    e.o << "    }\n    acc = gr_comb0(gr_comb0(acc, acc1), gr_comb0(acc2, acc3));\n  }\n";
    e.o << "  for (; j < " << je << "; ++j) {\n";   // at most one lane still has (fewer than four) elements
  } else {
    // one element per step of each of the workgroup's 256 threads: four steps written out with their
    // loads first, for the same reason as above; the accumulator takes the elements in the order of j
    const int STEP = 256;
    auto idx = [&](const std::string& su, const std::string& jx, const char* ind) {
      if (rank > kr) {
        e.o << ind << "long long jrem" << su << " = " << jx << ";\n";
        for (int k = rank - 1; k >= kr; --k) {
          if (k == kr) e.o << ind << "const long long i" << k << su << " = jrem" << su << ";\n";
          else e.o << ind << "const long long i" << k << su << " = gr_peel(jrem" << su << ", " << e.dim(k) << ");\n";
        }
      }
    };
    e.o << "  long long j = jbeg + threadIdx.x;\n  for (; j + " << 3 * STEP << " < jend; j += " << 4 * STEP << ") {\n";
    for (int u = 0; u < 4; ++u) {
      const std::string su = "_" + std::to_string(u);
      idx(su, "j + " + std::to_string(u * STEP), "    ");
      for (size_t i = 0; i < g.prog.size(); ++i) {
        const Instr& in = g.prog[i];
        if (in.kind != IKind::LOAD) continue;
        const AccessGroup& ag = g.groups[in.group];
        e.o << "    const " << cty(in.dtype) << " l" << i << su << " = p" << in.group << "[0";
        for (int k = 0; k < rank; ++k) {
          if (ag.structural_zero[k]) continue;
          if (k >= kr) e.o << " + (i" << k << su << " + " << in.delta[k] << ") * " << e.coef(in.group, k);
          else if (in.delta[k]) e.o << " + " << in.delta[k] << " * " << e.coef(in.group, k);
        }
        e.o << "];\n";
      }
    }
    e.o << "    __builtin_amdgcn_sched_barrier(0);\n";
    for (int u = 0; u < 4; ++u) {
      const std::string su = "_" + std::to_string(u);
      e.o << "    {\n";
      for (int k = rank - 1; k >= kr; --k) e.o << "      const long long i" << k << " = i" << k << su << "; (void)i" << k << ";\n";
      emit_scalar_program(e, g.prog, {ph.value}, [&](const Instr&, int id) { return "l" + std::to_string(id) + su; }, "0.0f", "t", "      ");
      e.o << "      acc = " << Em::combine(ph, "acc", "t" + std::to_string(ph.value)) << ";\n    }\n";
    }
    e.o << "  }\n  for (; j < jend; j += " << STEP << ") {\n";
  }
  if (rank > kr) {
    e.o << "    long long jrem = j;\n";
    for (int k = rank - 1; k >= kr; --k) {
      if (k == kr) e.o << "    const long long i" << k << " = jrem;\n";
      else e.o << "    const long long i" << k << " = gr_peel(jrem, " << e.dim(k) << ");\n";
    }
  }
  emit_scalar_program(e, g.prog, {ph.value},
                      [&](const Instr& in, int) {
                        const AccessGroup& ag = g.groups[in.group];
                        std::ostringstream s;
                        s << "p" << in.group << "[0";
                        for (int k = 0; k < rank; ++k) {
                          if (ag.structural_zero[k]) continue;
                          if (k >= kr) s << " + (i" << k << " + " << in.delta[k] << ") * " << e.coef(in.group, k);
                          else if (in.delta[k]) s << " + " << in.delta[k] << " * " << e.coef(in.group, k);
                        }
                        s << "]";
                        return s.str();
                      },
                      "0.0f", "t", "    ");
  e.o << "    acc = " << Em::combine(ph, "acc", "t" + std::to_string(ph.value)) << ";\n  }\n";
  e.o << "  GM " << T << "* const dst = NSPLIT > 1 ? (GM " << T << "*)" << e.slot(e.L.extra + 2) << " + split * NOUT : (GM " << T << "*)" << e.slot(e.L.out) << ";\n";
  e.o << "  acc = gr_lanes0(acc);\n"
         "  " << T << "* const sm = (" << T << "*)gr_sm;\n"
         "  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = acc;\n"
         "  __syncthreads();\n"
         "  acc = gr_comb0(gr_comb0(sm[0], sm[1]), gr_comb0(sm[2], sm[3]));\n"
         "  if (threadIdx.x == 0) dst[o] = acc;\n}\n";
  reduce_combine(e);
}

// ---- SCAN (map-scan) ------------------------------------------------------------

// Inclusive scan of the mapped values along the last iteration dimension.
//   mode 0: the scanned axis is contiguous.  A workgroup walks one chunk of one line in tiles
//           of 1024 elements: four elements per lane, a shuffle scan across the wave, 32 bytes
//           of LDS across the four waves, a running carry between tiles.  Lines longer than
//           one chunk take three kernels: chunk totals, an exclusive scan of the totals, the
//           chunks again with their offsets (reduce-then-scan).
//   mode 1: a thread per line, sequential along the axis (consecutive threads touch
//           consecutive addresses when an inner dimension is contiguous).
void gen_scan(Em& e) {
  const GroupPlan& g = e.g;
  const int rank = g.rank, sd = rank - 1;
  const Phase& ph = g.phases[0];
  const char* TA = cty(ph.out_dtype);  // accumulator = output type (f32, i32 for extrema, i64 for i32 sums)
  prelude(e);
  phase_helpers(e, 0, 64);
  e.o << "static __device__ __forceinline__ float gr_up(float v, int d) { return __shfl_up(v, d, 64); }\n"
         "static __device__ __forceinline__ int gr_up(int v, int d) { return __shfl_up(v, d, 64); }\n"
         "static __device__ __forceinline__ long long gr_up(long long v, int d) {\n"
         "  int lo = __shfl_up((int)(v & 0xffffffffll), d, 64), hi = __shfl_up((int)(v >> 32), d, 64);\n"
         "  return ((long long)hi << 32) | (unsigned int)lo;\n}\n";
  if (ph.out_dtype == GR_I64) e.o << "typedef long long l2 __attribute__((ext_vector_type(2)));\ntypedef l2 l2u __attribute__((aligned(8)));\n";
  const std::string ident = Em::identity(ph);
  auto conv = [&](const std::string& x) { return ph.out_dtype == GR_I64 && ph.in_dtype == GR_I32 ? "(long long)" + x : x; };
  auto load_at = [&](const std::string& col) {
    return [&e, &g, sd, col](const Instr& in, int) {
      const AccessGroup& ag = g.groups[in.group];
      std::ostringstream s;
      s << "p" << in.group << "[0";
      for (int k = 0; k < sd; ++k) if (!ag.structural_zero[k] && in.delta[k]) s << " + " << in.delta[k] << " * " << e.coef(in.group, k);
      if (!ag.structural_zero[sd]) s << " + (" << col << " + " << in.delta[sd] << ") * " << e.coef(in.group, sd);
      s << "]";
      return s.str();
    };
  };
  // common head: line index -> pointers
  auto head = [&](int per_block_line) {
    // (the chunk-count slot of a one-pass scan carries the poll limit in its upper half)
    // (one-pass scans: the chunk slot carries, in its upper half, the tag that marks a cell as published by this launch)
    if (g.scan_mode == 2 || g.scan_mode == 3) e.o << "  const long long LINES = " << e.S(e.L.extra) << ", CH = " << e.S(e.L.extra + 1) << " & 0xffffffffll, NCHUNK = " << e.S(e.L.extra + 3) << " & 0xffffffffll;\n"
                                 "  const unsigned EPOCH = (unsigned)(" << e.slot(e.L.extra + 1) << " >> 32);\n";
    else e.o << "  const long long LINES = " << e.S(e.L.extra) << ", CH = " << e.S(e.L.extra + 1) << ", NCHUNK = " << e.S(e.L.extra + 3) << " & 0xffffffffll;\n";
    e.o << "  const long long L = " << e.dim(sd) << ";\n";
    if (per_block_line == 2) {
      // a workgroup per tile of W neighbouring lines: consecutive workgroups take neighbouring
      // column blocks, all tiles of one position along the axis before the next
      const int LX = g.BX, W = 4 * g.BX;
      e.o << "  const long long D = " << e.dim(sd - 1) << ", NCB = (D + " << W - 1 << ") / " << W << ", NCHAIN = (LINES / D) * NCB;\n"
             "  const long long chain = blockIdx.x % NCHAIN, chunk = blockIdx.x / NCHAIN;\n"
             "  const long long cb = chain % NCB;\n"
             "  const int lx = threadIdx.x % " << LX << ", ly = threadIdx.x / " << LX << ";\n"
             "  const bool colok = cb * " << W << " + lx * 4 < D;\n"
             "  const long long line = (chain / NCB) * D + (colok ? cb * " << W << " + lx * 4 : 0);\n";
    }
    else if (per_block_line == 3) e.o << "  const long long line = (long long)blockIdx.x * " << 256 / g.BX << " + threadIdx.x / " << g.BX << ";\n  if (line >= LINES) return;\n";
    else if (per_block_line) e.o << "  const long long line = blockIdx.x / NCHUNK, chunk = blockIdx.x % NCHUNK;\n";
    else if (g.scan_vec) e.o << "  const long long gt = (long long)blockIdx.x * 256 + threadIdx.x;\n  if (gt >= (LINES / 4) * NCHUNK) return;\n"
                "  const long long line = 4 * (gt % (LINES / 4)), chunk = gt / (LINES / 4);\n  (void)chunk;\n";  // four lines per thread
    else e.o << "  const long long gt = (long long)blockIdx.x * 256 + threadIdx.x;\n  if (gt >= LINES * NCHUNK) return;\n"
                "  const long long line = gt % LINES, chunk = gt / LINES;\n  (void)chunk;\n";  // neighbouring threads: neighbouring lines
    e.o << "  long long lrem = line;\n";
    for (int k = sd - 1; k >= 0; --k) {
      if (k == 0) e.o << "  const long long i0 = lrem;\n";
      else e.o << "  const long long i" << k << " = gr_peel(lrem, " << e.dim(k) << ");\n";
    }
    group_pointers(e, "  ");
    for (size_t gi = 0; gi < g.groups.size(); ++gi) {
      const AccessGroup& ag = g.groups[gi];
      e.o << "  const GM " << cty(ag.dtype) << "* const p" << gi << " = q" << gi;
      for (int k = 0; k < sd; ++k) if (!ag.structural_zero[k]) e.o << " + i" << k << " * " << e.coef((int)gi, k);
      e.o << ";\n";
    }
    e.o << "  GM " << TA << "* const po = (GM " << TA << "*)" << e.slot(e.L.out);
    for (int k = 0; k < sd; ++k) e.o << " + i" << k << " * " << e.S(e.L.ocoef + k);
    e.o << ";\n";
    e.o << "  GM " << TA << "* const ws = (GM " << TA << "*)" << e.slot(e.L.extra + 2) << ";\n  (void)ws; (void)CH; (void)po; (void)L;\n";
  };

  // mode 0: the four elements a lane owns in a tile, fetched with one dwordx4 where the tile is
  // full (the scanned axis is contiguous for every access that follows it)
  auto tile_loads = [&](const std::string& ind) {
    for (size_t i = 0; i < g.prog.size(); ++i) {
      const Instr& in = g.prog[i];
      if (in.kind != IKind::LOAD) continue;
      const AccessGroup& ag = g.groups[in.group];
      std::ostringstream base;
      base << "p" << in.group;
      for (int k = 0; k < sd; ++k) if (!ag.structural_zero[k] && in.delta[k]) base << " + " << in.delta[k] << " * " << e.coef(in.group, k);
      e.o << ind << cty(in.dtype) << " l" << i << "[4];\n";
      if (ag.structural_zero[sd]) {
        e.o << ind << "for (int j = 0; j < 4; ++j) l" << i << "[j] = (" << base.str() << ")[0];\n";
      } else if (in.dtype == GR_I64) {
        e.o << ind << "for (int j = 0; j < 4; ++j) l" << i << "[j] = (c + j < cend) ? (" << base.str() << ")[c + j + " << in.delta[sd] << "] : 0;\n";
      } else {
        e.o << ind << "if (c + 4 <= cend) { const " << vty4(in.dtype) << " w = " << e.ld(in.group, vty4(in.dtype), base.str() + " + c + " + std::to_string(in.delta[sd]))
            << "; l" << i << "[0] = w[0]; l" << i << "[1] = w[1]; l" << i << "[2] = w[2]; l" << i << "[3] = w[3]; }\n";
        e.o << ind << "else { for (int j = 0; j < 4; ++j) l" << i << "[j] = (c + j < cend) ? (" << base.str() << ")[c + j + " << in.delta[sd] << "] : " << Em::zero(in.dtype) << "; }\n";
      }
    }
  };
  auto tile_value = [](const Instr&, int id) { return "l" + std::to_string(id) + "[j]"; };

  // ---- kernel 2 of 3 (both modes): exclusive scan of each line's chunk totals, in place (at most 4096 chunks): a workgroup per line, a lane per
  // line of many with few chunks (1352 x 15783 down the columns, 8 chunks: 13.6 us by workgroups, nearly all of it their launches, 4.8 by
  // lanes; the whole sum 70.0 and 61.2, of int32 1856 x 9173 72.5 and 64.5, 300 x 16381 27.2 and 18.2; up to 32 chunks, or for fewer lines, the loads of a lane cost
  // more: 1000 x 1001, 32 chunks, 11.3 by workgroups, 16.5 by lanes).  The additions of a lane are those of the workgroup, in the same order.
  auto offsets_kernel = [&]() {
    kernel_head(e, "gr_scan_offsets");
    e.o << "  const long long NCHUNK = " << e.S(e.L.extra + 3) << ";\n";
    e.o << "  if (NCHUNK <= " << kScanFewChunks << " && " << e.S(e.L.extra) << " >= " << kScanManyLines << ") {\n    const long long line = (long long)blockIdx.x * 256 + threadIdx.x;\n    if (line >= " << e.S(e.L.extra) << ") return;\n"
        << "    GM " << TA << "* const wl = (GM " << TA << "*)" << e.slot(e.L.extra + 2) << " + line * NCHUNK;\n    const int n = (int)NCHUNK;\n    " << TA << " x[" << kScanFewChunks << "];\n"
        << "#pragma unroll\n    for (int u = 0; u < " << kScanFewChunks << "; ++u) x[u] = gr_comb0(" << ident << ", wl[u < n ? u : 0]);\n"
        << "#pragma unroll\n    for (int d = 1; d < " << kScanFewChunks << "; d *= 2)\n#pragma unroll\n      for (int u = " << kScanFewChunks - 1 << "; u >= d; --u) x[u] = gr_comb0(x[u - d], x[u]);\n"
        << "#pragma unroll\n    for (int u = 0; u < " << kScanFewChunks << "; ++u) if (u < n) wl[u] = gr_comb0(" << ident << ", u ? x[u ? u - 1 : 0] : " << ident << ");\n    return;\n  }\n";
    e.o << "  GM " << TA << "* const w = (GM " << TA << "*)" << e.slot(e.L.extra + 2) << " + (long long)blockIdx.x * NCHUNK;\n";
    e.o << "  __shared__ long long gr_sm[4];\n";
    e.o << "  const int per = (int)((NCHUNK + 255) / 256);\n  const long long c0 = (long long)threadIdx.x * per;\n";
    e.o << "  " << TA << " v[16];\n  " << TA << " tot = " << ident << ";\n";
    e.o << "  for (int u = 0; u < 16; ++u) { v[u] = (u < per && c0 + u < NCHUNK) ? w[c0 + u] : " << ident << "; tot = gr_comb0(tot, v[u]); }\n";
    e.o << "  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;\n  " << TA << " x = tot;\n";
    for (int d = 1; d < 64; d <<= 1) e.o << "  { const " << TA << " y = gr_up(x, " << d << "); if (lane >= " << d << ") x = gr_comb0(y, x); }\n";
    e.o << "  " << TA << "* sm = (" << TA << "*)gr_sm;\n  if (lane == 63) sm[wave] = x;\n  __syncthreads();\n";
    e.o << "  " << TA << " off = " << ident << ";\n  for (int q = 0; q < wave; ++q) off = gr_comb0(off, sm[q]);\n";
    e.o << "  " << TA << " ex = gr_up(x, 1);\n  if (lane == 0) ex = " << ident << ";\n  off = gr_comb0(off, ex);\n";
    e.o << "  for (int u = 0; u < 16; ++u) if (u < per && c0 + u < NCHUNK) { w[c0 + u] = off; off = gr_comb0(off, v[u]); }\n}\n";
  };

  // Mode 1 walks a line sequentially; the running value makes every step depend on the one before,
  // and in the scan kernel the store of a step may alias the next load as far as the compiler
  // knows, so left alone each step waits for its own load.  The steps are therefore taken U at a
  // time: all loads of a batch first, then the U combines (and stores); a scalar loop finishes
  // the chunk.
  const int U = g.prog.size() <= 16 ? 8 : (g.prog.size() <= 48 ? 4 : 2);
  if (g.scan_mode == 1 && g.scan_vec) {
    // four neighbouring lines per thread: one dwordx4 per array and step
    const int ld = sd - 1;
    auto loads = [&](const std::string& jx, const std::string& sfx, const std::string& ind) {
      for (size_t i = 0; i < g.prog.size(); ++i) {
        const Instr& in = g.prog[i];
        if (in.kind != IKind::LOAD) continue;
        const AccessGroup& ag = g.groups[in.group];
        std::ostringstream at;
        at << "p" << in.group << " + 0";
        for (int k = 0; k < sd; ++k) if (!ag.structural_zero[k] && in.delta[k]) at << " + " << in.delta[k] << (k == ld ? std::string("") : " * " + e.coef(in.group, k));
        if (!ag.structural_zero[sd]) at << " + (" << jx << " + " << in.delta[sd] << ") * " << e.coef(in.group, sd);
        if (ag.structural_zero[ld]) e.o << ind << "const " << cty(in.dtype) << " u" << i << sfx << " = (" << at.str() << ")[0];\n";
        else e.o << ind << "const " << vty4(in.dtype) << " w" << i << sfx << " = " << e.ld(in.group, vty4(in.dtype), at.str()) << ";\n";
      }
    };
    auto step = [&](const std::string& jx, const std::string& sfx, const std::string& ind, bool store) {
      for (int c4 = 0; c4 < 4; ++c4) {
        const std::string pre = "v" + std::to_string(c4) + sfx + "_";
        emit_scalar_program(e, g.prog, {ph.value},
                            [&](const Instr& in, int id) {
                              const AccessGroup& ag = g.groups[in.group];
                              if (ag.structural_zero[ld]) return "u" + std::to_string(id) + sfx;
                              return "w" + std::to_string(id) + sfx + "[" + std::to_string(c4) + "]";
                            },
                            "0.0f", pre, ind);
        e.o << ind << "acc" << c4 << " = " << Em::combine(ph, "acc" + std::to_string(c4), pre + std::to_string(ph.value)) << ";\n";
      }
      if (store) {
        if (ph.out_dtype == GR_I64)
          e.o << ind << "{ l2u ov; ov[0] = acc0; ov[1] = acc1; *(GM l2u*)(po + (" << jx << ") * ostep) = ov; ov[0] = acc2; ov[1] = acc3; *(GM l2u*)(po + (" << jx << ") * ostep + 2) = ov; }\n";
        else {
          const char* vt = ph.out_dtype == GR_F32 ? "f4u" : "i4u";
          e.o << ind << "{ " << vt << " ov; ov[0] = acc0; ov[1] = acc1; ov[2] = acc2; ov[3] = acc3; *(GM " << vt << "*)(po + (" << jx << ") * ostep) = ov; }\n";
        }
      }
    };
    auto walk = [&](bool store) {
      e.o << "  long long j = cbeg;\n  for (; j + " << U << " <= cend; j += " << U << ") {\n";
      for (int u = 0; u < U; ++u) loads("j + " + std::to_string(u), "_" + std::to_string(u), "    ");
      for (int u = 0; u < U; ++u) { e.o << "    {\n"; step("j + " + std::to_string(u), "_" + std::to_string(u), "      ", store); e.o << "    }\n"; }
      e.o << "  }\n  for (; j < cend; ++j) {\n";
      loads("j", "", "    ");
      step("j", "", "    ", store);
      e.o << "  }\n";
    };
    kernel_head(e, "gr_scan_sums");
    head(false);
    e.o << "  const long long cbeg = chunk * CH, cend = (cbeg + CH < L) ? cbeg + CH : L;\n  " << TA << " acc0 = " << ident << ", acc1 = acc0, acc2 = acc0, acc3 = acc0;\n";
    walk(false);
    e.o << "  ws[line * NCHUNK + chunk] = acc0; ws[(line + 1) * NCHUNK + chunk] = acc1; ws[(line + 2) * NCHUNK + chunk] = acc2; ws[(line + 3) * NCHUNK + chunk] = acc3;\n}\n";
    offsets_kernel();
    kernel_head(e, "gr_scan");
    head(false);
    e.o << "  const long long cbeg = chunk * CH, cend = (cbeg + CH < L) ? cbeg + CH : L;\n";
    e.o << "  const long long ostep = " << e.S(e.L.ocoef + sd) << ";\n";
    e.o << "  " << TA << " acc0 = " << ident << ", acc1 = acc0, acc2 = acc0, acc3 = acc0;\n";
    e.o << "  if (NCHUNK > 1) { acc0 = ws[line * NCHUNK + chunk]; acc1 = ws[(line + 1) * NCHUNK + chunk]; acc2 = ws[(line + 2) * NCHUNK + chunk]; acc3 = ws[(line + 3) * NCHUNK + chunk]; }\n";
    walk(true);
    e.o << "}\n";
    return;
  }
  if (g.scan_mode == 1) {
    // a thread per (line, chunk), sequential along the axis; with several chunks per line the same
    // three steps as in mode 0: chunk totals, exclusive scan of the totals, chunks with offsets
    auto walk = [&](bool store) {
      e.o << "  long long j = cbeg;\n  for (; j + " << U << " <= cend; j += " << U << ") {\n";
      // the loads of the whole batch first (a load's value is named <prefix><id>)
      for (int u = 0; u < U; ++u) {
        const std::string pre = "t" + std::to_string(u) + "_";
        for (size_t i = 0; i < g.prog.size(); ++i) {
          if (g.prog[i].kind != IKind::LOAD) continue;
          e.o << "    const " << cty(g.prog[i].dtype) << ' ' << pre << i << " = " << load_at("(j + " + std::to_string(u) + ")")(g.prog[i], (int)i) << ";\n";
        }
      }
      for (int u = 0; u < U; ++u) {
        const std::string pre = "t" + std::to_string(u) + "_";
        std::vector<char> have(g.prog.size(), 0);
        for (size_t i = 0; i < g.prog.size(); ++i) if (g.prog[i].kind == IKind::LOAD) have[i] = 1;
        e.o << "    {\n";
        emit_scalar_program(e, g.prog, {ph.value}, load_at("j"), "0.0f", pre, "      ", &have);
        e.o << "      acc = " << Em::combine(ph, "acc", pre + std::to_string(ph.value)) << ";\n";
        if (store) e.o << "      po[(j + " << u << ") * ostep] = acc;\n";
        e.o << "    }\n";
      }
      e.o << "  }\n  for (; j < cend; ++j) {\n";
      emit_scalar_program(e, g.prog, {ph.value}, load_at("j"), "0.0f", "t", "    ");
      e.o << "    acc = " << Em::combine(ph, "acc", "t" + std::to_string(ph.value)) << ";\n";
      if (store) e.o << "    po[j * ostep] = acc;\n";
      e.o << "  }\n";
    };
    kernel_head(e, "gr_scan_sums");
    head(false);
    e.o << "  const long long cbeg = chunk * CH, cend = (cbeg + CH < L) ? cbeg + CH : L;\n  " << TA << " acc = " << ident << ";\n";
    walk(false);
    e.o << "  ws[line * NCHUNK + chunk] = acc;\n}\n";
    offsets_kernel();
    kernel_head(e, "gr_scan");
    head(false);
    e.o << "  const long long cbeg = chunk * CH, cend = (cbeg + CH < L) ? cbeg + CH : L;\n";
    e.o << "  const long long ostep = " << e.S(e.L.ocoef + sd) << ";\n  " << TA << " acc = NCHUNK > 1 ? ws[line * NCHUNK + chunk] : " << ident << ";\n";
    walk(true);
    e.o << "}\n";
    return;
  }


  if (g.scan_mode == 3) {
    // ---- mode 3: a scan along a non-contiguous axis with few lines, in ONE pass over the input.
    // A workgroup owns a tile of R positions along the scanned axis by W = 4*BX neighbouring lines
    // (the innermost line dimension is contiguous): BX lanes across the lines, each with four of
    // them, LY = 256/BX lane groups along the axis, RPL consecutive positions per lane, one vector
    // load per array and position.  The tile stays in registers: every lane scans its positions,
    // the lane groups exchange their totals through LDS, the tile's totals (one per line) are
    // published, and the offsets come from the tiles before it on the same lines.  Tiles of a
    // chain (the same W lines) form groups of G; the last tile of a group also publishes the group's
    // totals.  A line's offset in tile k of group q is
    //     fold(totals of groups 0..q-1, then of the tiles of group q before k),
    // taken by 256/W lanes per line in a fixed interleaved pattern and combined in lane order, so
    // the association, and with it every float result, depends on the shape only.  Cells are
    // 8-byte words (valid bit, value) written and read with relaxed agent-scope atomics; waits are
    // bounded, and a workgroup that runs out of polls takes its offsets from the input itself, so
    // every wave terminates whatever order tiles are dispatched in.  A small kernel clears the
    // cells before every launch.
    const int LX = g.BX, W = 4 * LX, LY = 256 / LX, RPL = (int)(g.scan_chunk / LY), R = (int)g.scan_chunk, P = 256 / W;
    const int ld = sd - 1;
    const char* V4 = ph.out_dtype == GR_F32 ? "f4" : "i4";
    const std::string bits = ph.out_dtype == GR_F32 ? "__float_as_uint" : "(unsigned)";
    const std::string unbits = ph.out_dtype == GR_F32 ? "__uint_as_float" : "(int)";
    kernel_head(e, "gr_scan_clear");
    e.o << "  const long long LINES = " << e.S(e.L.extra) << ", G = " << e.S(e.L.extra + 1) << " & 0xffffffffll, NCHUNK = " << e.S(e.L.extra + 3) << " & 0xffffffffll;\n"
           "  const long long D = " << e.dim(ld) << ", NCHAIN = (LINES / D) * ((D + " << W - 1 << ") / " << W << ");\n"
           "  const long long n = NCHAIN * (NCHUNK + (NCHUNK + G - 1) / G) * " << W << ";\n"
           "  GM unsigned long long* const w = (GM unsigned long long*)" << e.slot(e.L.extra + 2) << ";\n"
           "  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;\n  if (i < n) w[i] = 0ull;\n}\n";
    e.o << "static __device__ __forceinline__ unsigned long long gr_poll(GM unsigned long long* p, unsigned& polls, const unsigned tag) {\n"
           "  unsigned long long w = __hip_atomic_load((unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);\n"
           "  while ((unsigned)(w >> 32) != tag && polls) { __builtin_amdgcn_s_sleep(2); --polls; w = __hip_atomic_load((unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }\n"
           "  return w;\n}\n";
    kernel_head(e, "gr_scan");
    head(2);
    e.o << "  const long long G = CH;\n";
    e.o << "  __shared__ " << V4 << " gr_sm[" << LY << "][" << LX << "];\n  __shared__ " << TA << " gr_part[256];\n  __shared__ " << TA << " gr_base[" << W << "];\n";
    e.o << "  const long long cbeg = chunk * " << R << ", j0 = cbeg + ly * " << RPL << ";\n";
    e.o << "  const long long ostep = " << e.S(e.L.ocoef + sd) << ";\n";
    e.o << "  " << TA << " v[" << RPL << "][4];\n";
    // the values of the mapped expression at position jx of the lane's four lines
    auto loads = [&](const std::string& jx, const std::string& sfx, const std::string& ind) {
      for (size_t i = 0; i < g.prog.size(); ++i) {
        const Instr& in = g.prog[i];
        if (in.kind != IKind::LOAD) continue;
        const AccessGroup& ag = g.groups[in.group];
        std::ostringstream at;
        at << "p" << in.group << " + 0";
        for (int k = 0; k < sd; ++k) if (!ag.structural_zero[k] && in.delta[k]) at << " + " << in.delta[k] << (k == ld ? std::string("") : " * " + e.coef(in.group, k));
        if (!ag.structural_zero[sd]) at << " + (" << jx << " + " << in.delta[sd] << ") * " << e.coef(in.group, sd);
        if (ag.structural_zero[ld]) e.o << ind << "const " << cty(in.dtype) << " u" << i << sfx << " = (" << at.str() << ")[0];\n";
        else e.o << ind << "const " << vty4(in.dtype) << " w" << i << sfx << " = " << e.ld(in.group, vty4(in.dtype), at.str()) << ";\n";
      }
    };
    auto values = [&](const std::string& sfx, const std::string& ind, const std::function<std::string(int)>& dst) {
      for (int c4 = 0; c4 < 4; ++c4) {
        const std::string pre = "t" + std::to_string(c4) + sfx + "_";
        emit_scalar_program(e, g.prog, {ph.value},
                            [&](const Instr& in, int id) {
                              const AccessGroup& ag = g.groups[in.group];
                              if (ag.structural_zero[ld]) return "u" + std::to_string(id) + sfx;
                              return "w" + std::to_string(id) + sfx + "[" + std::to_string(c4) + "]";
                            },
                            "0.0f", pre, ind);
        e.o << ind << dst(c4) << " = " << pre << ph.value << ";\n";
      }
    };
    // the whole tile first: RPL vector loads per array in flight per lane; a tile inside the array
    // takes straight-line code without bounds checks
    e.o << "  const bool whole = cbeg + " << R << " <= L && (cb + 1) * " << W << " <= D;\n";
    e.o << "  if (whole) {\n";
    for (int u = 0; u < RPL; ++u) loads("j0 + " + std::to_string(u), "_" + std::to_string(u), "    ");
    for (int u = 0; u < RPL; ++u) { e.o << "    {\n"; values("_" + std::to_string(u), "      ", [&](int c4) { return "v[" + std::to_string(u) + "][" + std::to_string(c4) + "]"; }); e.o << "    }\n"; }
    e.o << "  } else {\n#pragma unroll\n    for (int u = 0; u < " << RPL << "; ++u) {\n"
           "      v[u][0] = v[u][1] = v[u][2] = v[u][3] = " << ident << ";\n"
           "      if (colok && j0 + u < L) {\n";
    loads("j0 + u", "", "        ");
    values("", "        ", [&](int c4) { return "v[u][" + std::to_string(c4) + "]"; });
    e.o << "      }\n    }\n  }\n";
    // scan inside the tile: down a lane's positions, then the lane groups through LDS
    e.o << "#pragma unroll\n  for (int u = 1; u < " << RPL << "; ++u)\n#pragma unroll\n    for (int c = 0; c < 4; ++c) v[u][c] = gr_comb0(v[u - 1][c], v[u][c]);\n";
    e.o << "  { " << V4 << " t; t[0] = v[" << RPL - 1 << "][0]; t[1] = v[" << RPL - 1 << "][1]; t[2] = v[" << RPL - 1 << "][2]; t[3] = v[" << RPL - 1 << "][3]; gr_sm[ly][lx] = t; }\n"
           "  __syncthreads();\n";
    e.o << "  " << TA << " off[4] = {" << ident << ", " << ident << ", " << ident << ", " << ident << "};\n"
           "  for (int q = 0; q < ly; ++q) { const " << V4 << " t = gr_sm[q][lx];\n#pragma unroll\n    for (int c = 0; c < 4; ++c) off[c] = gr_comb0(off[c], t[c]); }\n";
    // publish the tile's totals, one cell per line
    e.o << "  const long long NGROUP = (NCHUNK + G - 1) / G, grp = chunk / G, gfirst = grp * G;\n"
           "  GM unsigned long long* const wq = (GM unsigned long long*)" << e.slot(e.L.extra + 2) << ";\n"
           "  GM unsigned long long* const wa = wq + chain * NCHUNK * " << W << ";\n"
           "  GM unsigned long long* const wg = wq + NCHAIN * NCHUNK * " << W << " + chain * NGROUP * " << W << ";\n"
           "  if (threadIdx.x < " << W << ") {\n    " << TA << " tot = " << ident << ";\n"
           "    for (int q = 0; q < " << LY << "; ++q) tot = gr_comb0(tot, ((" << TA << "*)gr_sm)[q * " << W << " + threadIdx.x]);\n"
           "    __hip_atomic_store((unsigned long long*)(wa + chunk * " << W << " + threadIdx.x), ((unsigned long long)EPOCH << 32) | " << bits << "(tot), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);\n  }\n"
           "  unsigned polls = (unsigned)(" << e.slot(e.L.extra + 3) << " >> 32);\n  int lost = 0;\n"
           "  if (chunk == gfirst + G - 1 && threadIdx.x < " << W << ") {\n"
           "    // last tile of a full group: the group's totals, for every later group\n"
           "    " << TA << " acc = " << ident << ";\n"
           "    for (long long q = gfirst; q < gfirst + G; q += 4) {\n      unsigned long long w[4];\n"
           "#pragma unroll\n      for (int b = 0; b < 4; ++b) w[b] = __hip_atomic_load((unsigned long long*)(wa + (q + b) * " << W << " + threadIdx.x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);\n"
           "#pragma unroll\n      for (int b = 0; b < 4; ++b) {\n"
           "        if ((unsigned)(w[b] >> 32) != EPOCH) w[b] = gr_poll(wa + (q + b) * " << W << " + threadIdx.x, polls, EPOCH);\n"
           "        if ((unsigned)(w[b] >> 32) == EPOCH) acc = gr_comb0(acc, " << unbits << "((unsigned)w[b])); else lost = 1;\n      }\n    }\n"
           "    if (!lost) __hip_atomic_store((unsigned long long*)(wg + grp * " << W << " + threadIdx.x), ((unsigned long long)EPOCH << 32) | " << bits << "(acc), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);\n"
           "  }\n"
           "  {\n    const int col = threadIdx.x % " << W << ", part = threadIdx.x / " << W << ";\n"
           "    const long long n = grp + (chunk - gfirst);\n    " << TA << " acc = " << ident << ";\n"
           "    // (four cells asked for at a time: their latencies overlap; combined in index order all the same)\n"
           "    for (long long i = part; i < n; i += " << 4 * P << ") {\n"
           "      GM unsigned long long* cell[4];\n      unsigned long long w[4];\n"
           "#pragma unroll\n      for (int b = 0; b < 4; ++b) {\n        const long long ib = i + b * " << P << ";\n"
           "        cell[b] = ib < grp ? wg + ib * " << W << " + col : wa + (gfirst + ib - grp) * " << W << " + col;\n"
           "        w[b] = ib < n ? __hip_atomic_load((unsigned long long*)cell[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;\n      }\n"
           "#pragma unroll\n      for (int b = 0; b < 4; ++b) if (i + b * " << P << " < n) {\n"
           "        if ((unsigned)(w[b] >> 32) != EPOCH) w[b] = gr_poll(cell[b], polls, EPOCH);\n"
           "        if ((unsigned)(w[b] >> 32) == EPOCH) acc = gr_comb0(acc, " << unbits << "((unsigned)w[b])); else lost = 1;\n      }\n    }\n"
           "    gr_part[threadIdx.x] = acc;\n  }\n";
    e.o << "  if (__syncthreads_or(lost)) {\n"
           "    // out of polls: the offsets straight from the input (everything before this tile on its lines)\n"
           "    " << TA << " acc[4] = {" << ident << ", " << ident << ", " << ident << ", " << ident << "};\n"
           "    if (colok) for (long long j = ly; j < cbeg; j += " << LY << ") {\n      " << TA << " x[4];\n";
    loads("j", "", "      ");
    values("", "      ", [&](int c4) { return "x[" + std::to_string(c4) + "]"; });
    e.o << "#pragma unroll\n      for (int c = 0; c < 4; ++c) acc[c] = gr_comb0(acc[c], x[c]);\n    }\n"
           "    { " << V4 << " t; t[0] = acc[0]; t[1] = acc[1]; t[2] = acc[2]; t[3] = acc[3]; gr_sm[ly][lx] = t; }\n"
           "    __syncthreads();\n"
           "    if (threadIdx.x < " << W << ") {\n      " << TA << " b = " << ident << ";\n"
           "      for (int q = 0; q < " << LY << "; ++q) b = gr_comb0(b, ((" << TA << "*)gr_sm)[q * " << W << " + threadIdx.x]);\n"
           "      gr_base[threadIdx.x] = b;\n    }\n"
           "  } else if (threadIdx.x < " << W << ") {\n    " << TA << " b = gr_part[threadIdx.x];\n";
    for (int q = 1; q < P; ++q) e.o << "    b = gr_comb0(b, gr_part[" << q * W << " + threadIdx.x]);\n";
    e.o << "    gr_base[threadIdx.x] = b;\n  }\n  __syncthreads();\n";
    e.o << "#pragma unroll\n  for (int c = 0; c < 4; ++c) off[c] = gr_comb0(gr_base[lx * 4 + c], off[c]);\n";
    {
      const char* vt = ph.out_dtype == GR_F32 ? "f4u" : "i4u";
      const std::string st = (g.nt & 8) ? "__builtin_nontemporal_store(ov, (GM " + std::string(vt) + "*)(po + (j0 + u) * ostep))" : "*(GM " + std::string(vt) + "*)(po + (j0 + u) * ostep) = ov";
      e.o << "  if (whole) {\n#pragma unroll\n    for (int u = 0; u < " << RPL << "; ++u) {\n"
             "      " << vt << " ov; for (int c = 0; c < 4; ++c) ov[c] = gr_comb0(off[c], v[u][c]); " << st << ";\n    }\n    return;\n  }\n";
      e.o << "#pragma unroll\n  for (int u = 0; u < " << RPL << "; ++u) {\n"
             "    if (colok && j0 + u < L) { " << vt << " ov; for (int c = 0; c < 4; ++c) ov[c] = gr_comb0(off[c], v[u][c]); " << st << "; }\n  }\n}\n";
    }
    return;
  }

  if (g.scan_mode == 2) {
    // ---- mode 2: long contiguous lines in ONE pass over the input.  A workgroup owns a tile of TU x 1024
    // consecutive elements of a line, keeps it in registers, scans it, publishes the tile's total and
    // needs, before it may store, the combination of everything before its tile.  Tiles form groups
    // of 128; the last tile of a group also publishes the group's total.  A tile's offset is
    //     fold(totals of the earlier groups) (+) fold(totals of the earlier tiles of its own group),
    // each fold taken lane by lane in a fixed pattern, so the association -- and with it every float
    // result -- does not depend on timing.  A published cell is one 8-byte word (valid bit, value)
    // written and read with relaxed agent-scope atomics.  Waiting is bounded: a workgroup that runs
    // out of polls computes its offset from the input itself, so every wave terminates whatever order
    // the tiles are dispatched in (in dispatch order, which is what happens, everything a tile waits
    // for is already running).  A small kernel clears the cells before every launch.
    const int TU = (int)(g.scan_chunk / 1024);  // blocks of 1024 elements per tile
    const std::string bits = ph.out_dtype == GR_F32 ? "__float_as_uint" : "(unsigned)";
    const std::string unbits = ph.out_dtype == GR_F32 ? "__uint_as_float" : "(int)";
    kernel_head(e, "gr_scan_clear");
    e.o << "  const long long LINES = " << e.S(e.L.extra) << ", NCHUNK = " << e.S(e.L.extra + 3) << " & 0xffffffffll;\n"
           "  const long long n = LINES * NCHUNK + LINES * ((NCHUNK + 127) / 128);\n"   // one cell per tile and per group
           "  GM unsigned long long* const w = (GM unsigned long long*)" << e.slot(e.L.extra + 2) << ";\n"
           "  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;\n  if (i < n) w[i] = 0ull;\n}\n";
    // wave-wide inclusive scan with row shifts inside rows of 16 lanes and two row broadcasts; lanes without a source take the identity
    e.o << "#define GR_DPP(idn, v, ctrl, rmask) " << unbits << "((unsigned)__builtin_amdgcn_update_dpp((int)" << bits << "(idn), (int)" << bits << "(v), ctrl, rmask, 0xf, false))\n";
    e.o << "static __device__ __forceinline__ " << TA << " gr_wscan(" << TA << " x) {\n  const " << TA << " idn = " << ident << ";\n"
           "  x = gr_comb0(GR_DPP(idn, x, 0x111, 0xf), x);\n  x = gr_comb0(GR_DPP(idn, x, 0x112, 0xf), x);\n"
           "  x = gr_comb0(GR_DPP(idn, x, 0x114, 0xf), x);\n  x = gr_comb0(GR_DPP(idn, x, 0x118, 0xf), x);\n"
           "  x = gr_comb0(GR_DPP(idn, x, 0x142, 0xa), x);\n  x = gr_comb0(GR_DPP(idn, x, 0x143, 0xc), x);\n  return x;\n}\n";
    e.o << "static __device__ __forceinline__ unsigned long long gr_poll(GM unsigned long long* p, unsigned& polls, const unsigned tag) {\n"
           "  unsigned long long w = __hip_atomic_load((unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);\n"
           "  while ((unsigned)(w >> 32) != tag && polls) { __builtin_amdgcn_s_sleep(8); --polls; w = __hip_atomic_load((unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }\n"
           "  return w;\n}\n";
    e.o << "static __device__ __forceinline__ " << TA << " gr_fold(" << TA << " x, " << TA << "* f) {\n"
           "  x = gr_lanes0(x);\n  if ((threadIdx.x & 63) == 0) f[threadIdx.x >> 6] = x;\n  __syncthreads();\n"
           "  return gr_comb0(gr_comb0(f[0], f[1]), gr_comb0(f[2], f[3]));\n}\n";
    kernel_head(e, "gr_scan");
    head(true);
    e.o << "  __shared__ " << TA << " gr_wt[" << TU << "][4];\n  __shared__ " << TA << " gr_fs[4][4];\n";
    e.o << "  const long long cbeg = chunk * CH;\n  const int clen = (int)((cbeg + CH < L) ? CH : L - cbeg);\n";
    e.o << "  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;\n";
    e.o << "  " << TA << " v[" << TU << "][4];\n";
    // positions inside the tile are 32-bit offsets from the tile's first element (one 64-bit base per array)
    for (size_t gi = 0; gi < g.groups.size(); ++gi)
      e.o << "  const GM " << cty(g.groups[gi].dtype) << "* const tp" << gi << " = p" << gi << (g.groups[gi].structural_zero[sd] ? "" : " + cbeg") << ";\n";
    e.o << "  GM " << TA << "* const tpo = po + cbeg;\n";
    // the whole tile first: TU vector loads per array in flight per lane
    // (a full tile -- every tile of a line but the last -- takes straight-line code without bounds checks)
    e.o << "  const bool whole = clen == " << TU * 1024 << ";\n";
    e.o << "  if (whole) {\n    const int cend = " << TU * 1024 << ";\n";
    for (size_t gi = 0; gi < g.groups.size(); ++gi) e.o << "    const GM " << cty(g.groups[gi].dtype) << "* const p" << gi << " = tp" << gi << ";\n";
    e.o << "#pragma unroll\n    for (int u = 0; u < " << TU << "; ++u) {\n      const int c = u * 1024 + threadIdx.x * 4;\n";
    tile_loads("      ");
    e.o << "#pragma unroll\n      for (int j = 0; j < 4; ++j) {\n";
    emit_scalar_program(e, g.prog, {ph.value}, tile_value, "0.0f", "t", "        ");
    e.o << "        v[u][j] = " << conv("t" + std::to_string(ph.value)) << ";\n      }\n    }\n  } else {\n    const int cend = clen;\n";
    for (size_t gi = 0; gi < g.groups.size(); ++gi) e.o << "    const GM " << cty(g.groups[gi].dtype) << "* const p" << gi << " = tp" << gi << ";\n";
    e.o << "#pragma unroll\n    for (int u = 0; u < " << TU << "; ++u) {\n      const int c = u * 1024 + threadIdx.x * 4;\n";
    tile_loads("      ");
    e.o << "#pragma unroll\n      for (int j = 0; j < 4; ++j) {\n        v[u][j] = " << ident << ";\n        if (c + j < cend) {\n";
    emit_scalar_program(e, g.prog, {ph.value}, tile_value, "0.0f", "t", "          ");
    e.o << "          v[u][j] = " << conv("t" + std::to_string(ph.value)) << ";\n        }\n      }\n    }\n  }\n";
    // scan inside the tile: four elements of a lane, the lanes of a wave, then waves and blocks through LDS
    e.o << "  " << TA << " xs[" << TU << "];\n";
    e.o << "#pragma unroll\n  for (int u = 0; u < " << TU << "; ++u) {\n"
           "    v[u][1] = gr_comb0(v[u][0], v[u][1]); v[u][2] = gr_comb0(v[u][1], v[u][2]); v[u][3] = gr_comb0(v[u][2], v[u][3]);\n"
           "    xs[u] = gr_wscan(v[u][3]);\n    if (lane == 63) gr_wt[u][wave] = xs[u];\n  }\n  __syncthreads();\n";
    e.o << "  " << TA << " carry = " << ident << ";\n";
    e.o << "#pragma unroll\n  for (int u = 0; u < " << TU << "; ++u) {\n    " << TA << " b = carry;\n"
           "    for (int q = 0; q < wave; ++q) b = gr_comb0(b, gr_wt[u][q]);\n"
           "    { const " << TA << " ex = GR_DPP(" << ident << ", xs[u], 0x138, 0xf); if (lane != 0) b = gr_comb0(b, ex); }\n"
           "#pragma unroll\n    for (int j = 0; j < 4; ++j) v[u][j] = gr_comb0(b, v[u][j]);\n"
           "    carry = gr_comb0(carry, gr_comb0(gr_comb0(gr_wt[u][0], gr_wt[u][1]), gr_comb0(gr_wt[u][2], gr_wt[u][3])));\n  }\n";
    // publish, then collect the offset
    e.o << "  const long long NGROUP = (NCHUNK + 127) / 128, grp = chunk / 128, gfirst = grp * 128;\n"
           "  GM unsigned long long* const wq = (GM unsigned long long*)" << e.slot(e.L.extra + 2) << ";\n"
           "  GM unsigned long long* const wa = wq + line * NCHUNK;\n"
           "  GM unsigned long long* const wg = wq + LINES * NCHUNK + line * NGROUP;\n"
           "  if (threadIdx.x == 0) __hip_atomic_store((unsigned long long*)(wa + chunk), ((unsigned long long)EPOCH << 32) | " << bits << "(carry), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);\n"
           "  unsigned polls = (unsigned)(" << e.slot(e.L.extra + 3) << " >> 32);\n  int lost = 0;\n"
           "  if (chunk == gfirst + 127) {\n"
           "    // last tile of a full group: the group's total, for every later group\n"
           "    " << TA << " acc = " << ident << ";\n"
           "    if (threadIdx.x < 128) { const unsigned long long w = gr_poll(wa + gfirst + threadIdx.x, polls, EPOCH); if ((unsigned)(w >> 32) == EPOCH) acc = " << unbits << "((unsigned)w); else lost = 1; }\n"
           "    const " << TA << " tot = gr_fold(acc, gr_fs[0]);\n"
           "    if (!__syncthreads_or(lost) && threadIdx.x == 0) __hip_atomic_store((unsigned long long*)(wg + grp), ((unsigned long long)EPOCH << 32) | " << bits << "(tot), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);\n"
           "  }\n"
           "  " << TA << " p1 = " << ident << ", p2 = " << ident << ";\n"
           "  // (first the earlier groups, then the earlier tiles of this group: measured faster than waiting for both at once)\n"
           "  for (long long q = threadIdx.x; q < grp; q += 256) { const unsigned long long w = gr_poll(wg + q, polls, EPOCH); if ((unsigned)(w >> 32) == EPOCH) p1 = gr_comb0(p1, " << unbits << "((unsigned)w)); else lost = 1; }\n"
           "  for (long long q = gfirst + threadIdx.x; q < chunk; q += 256) { const unsigned long long w = gr_poll(wa + q, polls, EPOCH); if ((unsigned)(w >> 32) == EPOCH) p2 = gr_comb0(p2, " << unbits << "((unsigned)w)); else lost = 1; }\n"
           "  p1 = gr_fold(p1, gr_fs[1]);\n  p2 = gr_fold(p2, gr_fs[2]);\n"
           "  " << TA << " base = gr_comb0(p1, p2);\n"
           "  if (__syncthreads_or(lost)) {\n"
           "    // out of polls: the offset straight from the input (the whole line before this tile)\n"
           "    " << TA << " acc = " << ident << ";\n    const long long cend = cbeg;\n"
           "    for (long long t0 = 0; t0 < cbeg; t0 += 1024) {\n      const long long c = t0 + threadIdx.x * 4;\n";
    tile_loads("      ");
    e.o << "#pragma unroll\n      for (int j = 0; j < 4; ++j) {\n        if (c + j < cend) {\n";
    emit_scalar_program(e, g.prog, {ph.value}, tile_value, "0.0f", "t", "          ");
    e.o << "          acc = " << Em::combine(ph, "acc", "t" + std::to_string(ph.value)) << ";\n        }\n      }\n    }\n"
           "    base = gr_fold(acc, gr_fs[3]);\n  }\n";
    {
      const char* vt = ph.out_dtype == GR_F32 ? "f4u" : "i4u";
      const std::string st = (g.nt & 8) ? "__builtin_nontemporal_store(ov, (GM " + std::string(vt) + "*)(tpo + c))" : "*(GM " + std::string(vt) + "*)(tpo + c) = ov";
      e.o << "  if (whole) {\n#pragma unroll\n    for (int u = 0; u < " << TU << "; ++u) {\n      const int c = u * 1024 + threadIdx.x * 4;\n"
             "      " << vt << " ov; for (int j = 0; j < 4; ++j) ov[j] = gr_comb0(base, v[u][j]); " << st << ";\n    }\n    return;\n  }\n";
    }
    e.o << "#pragma unroll\n  for (int u = 0; u < " << TU << "; ++u) {\n    const int c = u * 1024 + threadIdx.x * 4;\n";
    {
      const char* vt = ph.out_dtype == GR_F32 ? "f4u" : "i4u";
      e.o << "    if (c + 4 <= clen) { " << vt << " ov; for (int j = 0; j < 4; ++j) ov[j] = gr_comb0(base, v[u][j]); "
          << ((g.nt & 8) ? "__builtin_nontemporal_store(ov, (GM " + std::string(vt) + "*)(tpo + c))" : "*(GM " + std::string(vt) + "*)(tpo + c) = ov") << "; }\n"
             "    else { for (int j = 0; j < 4; ++j) if (c + j < clen) tpo[c + j] = gr_comb0(base, v[u][j]); }\n  }\n}\n";
    }
    return;
  }

  if (g.scan_mode == 4) {
    // ---- mode 4: short contiguous lines, LG = 16 or 64 lanes each, several lines to a workgroup and no barrier.  A line is
    // NP positions of four elements per lane, all loaded at once; the last position, which may stick out of the line, is
    // loaded from the line's last four elements and shifted into place.  Each position is scanned across its lanes with
    // row shifts (and row broadcasts for 64 lanes); the positions' totals are combined in a tree.  Bound by HBM.
    const int LG = g.BX, NP = g.NP;
    const bool wide = ph.out_dtype == GR_I64;
    const std::string bits = ph.out_dtype == GR_F32 ? "__float_as_uint" : "(unsigned)";
    const std::string unbits = ph.out_dtype == GR_F32 ? "__uint_as_float" : "(int)";
    if (wide)
      e.o << "#define GR_DPP(idn, v, ctrl, rmask) ((long long)(((unsigned long long)(unsigned)__builtin_amdgcn_update_dpp((int)((idn) >> 32), (int)((v) >> 32), ctrl, rmask, 0xf, false) << 32) | "
             "(unsigned)__builtin_amdgcn_update_dpp((int)(idn), (int)(v), ctrl, rmask, 0xf, false)))\n";
    else e.o << "#define GR_DPP(idn, v, ctrl, rmask) " << unbits << "((unsigned)__builtin_amdgcn_update_dpp((int)" << bits << "(idn), (int)" << bits << "(v), ctrl, rmask, 0xf, false))\n";
    e.o << "static __device__ __forceinline__ " << TA << " gr_gscan(" << TA << " x) {\n  const " << TA << " idn = " << ident << ";\n"
           "  x = gr_comb0(GR_DPP(idn, x, 0x111, 0xf), x);\n  x = gr_comb0(GR_DPP(idn, x, 0x112, 0xf), x);\n"
           "  x = gr_comb0(GR_DPP(idn, x, 0x114, 0xf), x);\n  x = gr_comb0(GR_DPP(idn, x, 0x118, 0xf), x);\n";
    if (LG == 64) e.o << "  x = gr_comb0(GR_DPP(idn, x, 0x142, 0xa), x);\n  x = gr_comb0(GR_DPP(idn, x, 0x143, 0xc), x);\n";
    e.o << "  return x;\n}\n";
    if (wide)
      e.o << "static __device__ __forceinline__ long long gr_bc(long long v, int l) {\n"
             "  const int lo = __shfl((int)(v & 0xffffffffll), l, 64), hi = __shfl((int)(v >> 32), l, 64);\n  return ((long long)hi << 32) | (unsigned int)lo;\n}\n";
    else e.o << "static __device__ __forceinline__ " << TA << " gr_bc(" << TA << " v, int l) { return __shfl(v, l, 64); }\n";
    kernel_head(e, "gr_scan");
    head(3);
    e.o << "  const int lane = threadIdx.x & " << LG - 1 << ", last = (threadIdx.x & 63) | " << LG - 1 << ", c0 = lane * 4, n = (int)L;\n";
    const std::string clast = "(c0 + " + std::to_string((NP - 1) * LG * 4) + ")";
    e.o << "  const int cl = " << clast << " + 4 <= n ? " << clast << " : n - 4, sh = " << clast << " - cl;\n";
    for (int p = 0; p < NP; ++p) {
      const std::string sp = std::to_string(p), at = p + 1 < NP ? "c0 + " + std::to_string(p * LG * 4) : std::string("cl");
      for (size_t i = 0; i < g.prog.size(); ++i) {
        const Instr& in = g.prog[i];
        if (in.kind != IKind::LOAD) continue;
        const AccessGroup& ag = g.groups[in.group];
        std::ostringstream base;
        base << "p" << in.group;
        for (int k = 0; k < sd; ++k) if (!ag.structural_zero[k] && in.delta[k]) base << " + " << in.delta[k] << " * " << e.coef(in.group, k);
        if (ag.structural_zero[sd]) { if (p == 0) e.o << "  const " << cty(in.dtype) << " u" << i << " = (" << base.str() << ")[0];\n"; }
        else e.o << "  const " << vty4(in.dtype) << " w" << i << "_" << sp << " = " << e.ld(in.group, vty4(in.dtype), base.str() + " + " + at + " + " + std::to_string(in.delta[sd])) << ";\n";
      }
    }
    e.o << "  __builtin_amdgcn_sched_barrier(0);\n";
    for (int p = 0; p < NP; ++p) {
      const std::string sp = std::to_string(p);
      e.o << "  " << TA << " v" << sp << "[4];\n";
      for (int j = 0; j < 4; ++j) {
        const std::string pre = "t" + std::to_string(j) + "_";
        e.o << "  {\n";
        emit_scalar_program(e, g.prog, {ph.value},
                            [&](const Instr& in, int id) { return g.groups[in.group].structural_zero[sd] ? "u" + std::to_string(id) : "w" + std::to_string(id) + "_" + sp + "[" + std::to_string(j) + "]"; },
                            "0.0f", pre, "    ");
        e.o << "    v" << sp << "[" << j << "] = " << conv(pre + std::to_string(ph.value)) << ";\n  }\n";
      }
      if (p + 1 == NP) {
        // into place: elements sh .. 3 move to the front, the rest lies behind the line's end
        e.o << "  if (sh) {\n    const " << TA << " a1 = v" << sp << "[1], a2 = v" << sp << "[2], a3 = v" << sp << "[3];\n"
               "    v" << sp << "[0] = sh == 1 ? a1 : sh == 2 ? a2 : sh == 3 ? a3 : " << ident << ";\n"
               "    v" << sp << "[1] = sh == 1 ? a2 : sh == 2 ? a3 : " << ident << ";\n"
               "    v" << sp << "[2] = sh == 1 ? a3 : " << ident << ";\n    v" << sp << "[3] = " << ident << ";\n  }\n";
      }
      e.o << "  for (int j = 1; j < 4; ++j) v" << sp << "[j] = gr_comb0(v" << sp << "[j - 1], v" << sp << "[j]);\n"
             "  const " << TA << " x" << sp << " = gr_gscan(v" << sp << "[3]);\n";
      if (p + 1 < NP) e.o << "  const " << TA << " s" << sp << "_0 = gr_bc(x" << sp << ", last);\n";
    }
    // inclusive scan of the positions' totals, log2(NP) combines deep
    int level = 0;
    for (int d = 1; d < NP - 1; d *= 2, ++level)
      for (int p = 0; p + 1 < NP; ++p) {
        const std::string lv = "_" + std::to_string(level);
        e.o << "  const " << TA << " s" << p << "_" << level + 1 << " = " << (p >= d ? "gr_comb0(s" + std::to_string(p - d) + lv + ", s" + std::to_string(p) + lv + ")" : "s" + std::to_string(p) + lv) << ";\n";
      }
    for (int p = 0; p < NP; ++p) {
      const std::string sp = std::to_string(p), c = "c0 + " + std::to_string(p * LG * 4);
      e.o << "  {\n    const " << TA << " idn = " << ident << ", ex = GR_DPP(idn, x" << sp << ", " << (LG == 64 ? "0x138" : "0x111") << ", 0xf), b = "
          << (p ? "lane ? gr_comb0(s" + std::to_string(p - 1) + "_" + std::to_string(level) + ", ex) : s" + std::to_string(p - 1) + "_" + std::to_string(level) : std::string("ex")) << ";\n"
             "    if (" << (p == 0 ? "lane" : "true") << ") for (int j = 0; j < 4; ++j) v" << sp << "[j] = gr_comb0(b, v" << sp << "[j]);\n    const int c = " << c << ";\n    ";
      if (p + 1 == NP) e.o << "if (c + 4 <= n) ";
      if (wide) e.o << "{ l2u ov; ov[0] = v" << sp << "[0]; ov[1] = v" << sp << "[1]; *(GM l2u*)(po + c) = ov; ov[0] = v" << sp << "[2]; ov[1] = v" << sp << "[3]; *(GM l2u*)(po + c + 2) = ov; }\n";
      else {
        const std::string vt = ph.out_dtype == GR_F32 ? "f4u" : "i4u";
        e.o << "{ " << vt << " ov; for (int j = 0; j < 4; ++j) ov[j] = v" << sp << "[j]; " << ((g.nt & 8) ? "__builtin_nontemporal_store(ov, (GM " + vt + "*)(po + c))" : "*(GM " + vt + "*)(po + c) = ov") << "; }\n";
      }
      if (p + 1 == NP) e.o << "    else { if (c < n) po[c] = v" << sp << "[0]; if (c + 1 < n) po[c + 1] = v" << sp << "[1]; if (c + 2 < n) po[c + 2] = v" << sp << "[2]; }\n";
      e.o << "  }\n";
    }
    e.o << "}\n";
    return;
  }

  // ---- mode 0, kernel 1 of 3: chunk totals (only launched when a line has several chunks)
  kernel_head(e, "gr_scan_sums");
  head(true);
  e.o << "  __shared__ long long gr_sm[4];\n";
  e.o << "  const long long cbeg = chunk * CH, cend = (cbeg + CH < L) ? cbeg + CH : L;\n  " << TA << " acc = " << ident << ";\n";
  e.o << "  for (long long t0 = cbeg; t0 < cend; t0 += 1024) {\n    const long long c = t0 + threadIdx.x * 4;\n";
  tile_loads("    ");
  e.o << "#pragma unroll\n    for (int j = 0; j < 4; ++j) {\n      if (c + j < cend) {\n";
  emit_scalar_program(e, g.prog, {ph.value}, tile_value, "0.0f", "t", "        ");
  e.o << "        acc = " << Em::combine(ph, "acc", "t" + std::to_string(ph.value)) << ";\n      }\n    }\n  }\n";
  e.o << "  acc = gr_lanes0(acc);\n  { " << TA << "* sm = (" << TA << "*)gr_sm;\n    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = acc;\n    __syncthreads();\n"
         "    if (threadIdx.x == 0) ws[line * NCHUNK + chunk] = gr_comb0(gr_comb0(sm[0], sm[1]), gr_comb0(sm[2], sm[3])); }\n}\n";

  offsets_kernel();

  // ---- kernel 3 of 3 (the only one for single-chunk lines): scan of a chunk with its offset
  kernel_head(e, "gr_scan");
  head(true);
  e.o << "  __shared__ long long gr_sm[2][4];\n";
  e.o << "  const long long cbeg = chunk * CH, cend = (cbeg + CH < L) ? cbeg + CH : L;\n";
  e.o << "  " << TA << " carry = NCHUNK > 1 ? ws[line * NCHUNK + chunk] : " << ident << ";\n";
  e.o << "  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;\n  int buf = 0;\n";
  e.o << "  for (long long t0 = cbeg; t0 < cend; t0 += 1024) {\n    const long long c = t0 + threadIdx.x * 4;\n    " << TA << " v[4];\n";
  tile_loads("    ");
  e.o << "#pragma unroll\n    for (int j = 0; j < 4; ++j) {\n      v[j] = " << ident << ";\n      if (c + j < cend) {\n";
  emit_scalar_program(e, g.prog, {ph.value}, tile_value, "0.0f", "t", "        ");
  e.o << "        v[j] = " << conv("t" + std::to_string(ph.value)) << ";\n      }\n    }\n";
  e.o << "    v[1] = gr_comb0(v[0], v[1]); v[2] = gr_comb0(v[1], v[2]); v[3] = gr_comb0(v[2], v[3]);\n    " << TA << " x = v[3];\n";
  for (int d = 1; d < 64; d <<= 1) e.o << "    { const " << TA << " y = gr_up(x, " << d << "); if (lane >= " << d << ") x = gr_comb0(y, x); }\n";
  e.o << "    " << TA << "* sm = (" << TA << "*)gr_sm[buf];\n    if (lane == 63) sm[wave] = x;\n    __syncthreads();\n";
  e.o << "    " << TA << " base = carry;\n    for (int q = 0; q < wave; ++q) base = gr_comb0(base, sm[q]);\n";
  e.o << "    { " << TA << " ex = gr_up(x, 1); if (lane != 0) base = gr_comb0(base, ex); }\n";
  if (ph.out_dtype == GR_I64)
    e.o << "    if (c + 4 <= cend) { l2u ov; for (int j = 0; j < 2; ++j) ov[j] = gr_comb0(base, v[j]); *(GM l2u*)(po + c) = ov; for (int j = 0; j < 2; ++j) ov[j] = gr_comb0(base, v[j + 2]); *(GM l2u*)(po + c + 2) = ov; }\n"
           "    else { for (int j = 0; j < 4; ++j) if (c + j < cend) po[c + j] = gr_comb0(base, v[j]); }\n";
  else {
    const char* vt = ph.out_dtype == GR_F32 ? "f4u" : "i4u";
    e.o << "    if (c + 4 <= cend) { " << vt << " ov; for (int j = 0; j < 4; ++j) ov[j] = gr_comb0(base, v[j]); "
        << ((g.nt & 8) ? "__builtin_nontemporal_store(ov, (GM " + std::string(vt) + "*)(po + c))" : "*(GM " + std::string(vt) + "*)(po + c) = ov") << "; }\n"
           "    else { for (int j = 0; j < 4; ++j) if (c + j < cend) po[c + j] = gr_comb0(base, v[j]); }\n";
  }
  e.o << "    carry = gr_comb0(carry, gr_comb0(gr_comb0(sm[0], sm[1]), gr_comb0(sm[2], sm[3])));\n    buf ^= 1;\n  }\n}\n";
}

// ---- GEMV -----------------------------------------------------------------------

// Epilogue: the pointwise consumers of the dot, evaluated at output index `idx`.
void gemv_epilogue(Em& e, const std::string& idx, const std::string& acc, const std::string& indent) {
  const GroupPlan& g = e.g;
  emit_scalar_program(e, g.prog, g.results,
                      [&](const Instr& in, int) {
                        const AccessGroup& ag = g.groups[in.group];
                        if (ag.structural_zero[0]) return e.qp + std::to_string(in.group) + "[0]";
                        return e.qp + std::to_string(in.group) + "[(" + idx + " + " + std::to_string(in.delta[0]) + ") * " + e.coef(in.group, 0) + "]";
                      },
                      acc, "t", indent);
}

void gen_gemv_rowdot(Em& e) {
  const GroupPlan& g = e.g;
  const int LPR = g.LPR, KV = g.KV, RPB = 256 / LPR;
  const AccessGroup& mg = g.groups[g.mat_group];
  const AccessGroup& vg = g.groups[g.vec_group];
  const bool mat_unit = mg.coef[1] == 1, vec_unit = vg.coef[1] == 1;
  prelude(e);
  kernel_head(e, kernel_name(g));
  e.o << "  const long long M = " << e.S(e.L.extra) << ", K = " << e.S(e.L.extra + 1) << ";\n";
  group_pointers(e, "  ");
  e.o << "  const GM float* const A = q" << g.mat_group << "; const GM float* const V = q" << g.vec_group << ";\n";
  e.o << "  const long long am = " << e.coef(g.mat_group, 0) << ", ak = " << (mat_unit ? std::string("1") : e.coef(g.mat_group, 1))
      << ", vk = " << (vec_unit ? std::string("1") : e.coef(g.vec_group, 1)) << ";\n";
  e.o << "  const int lane = threadIdx.x % " << LPR << ", rib = threadIdx.x / " << LPR << ";\n";
  e.o << "  GM float* const out = (GM float*)" << e.slot(e.L.out) << ";\n";
  const int CH = LPR * 4;  // k elements per chunk of one row
  // one pass if the whole row fits KV chunks, else loop over groups of KV chunks
  e.o << "  const bool single = K <= " << (long long)CH * KV << ";\n";
  e.o << "  float wv[" << KV << "][4];\n";
  e.o << "  if (single) {\n#pragma unroll\n    for (int q = 0; q < " << KV << "; ++q) {\n      const long long k0 = (long long)q * " << CH << " + lane * 4;\n";
  e.o << "      for (int j = 0; j < 4; ++j) wv[q][j] = (k0 + j < K) ? V[(k0 + j) * vk] : 0.0f;\n    }\n  }\n";
  e.o << "  for (long long row = (long long)blockIdx.x * " << RPB << " + rib; row < M; row += (long long)gridDim.x * " << RPB << ") {\n";
  e.o << "    const GM float* const Ar = A + row * am;\n    float acc = 0.0f;\n";
  e.o << "    if (single) {\n";
  e.o << "      float xv[" << KV << "][4];\n#pragma unroll\n      for (int q = 0; q < " << KV << "; ++q) {\n        const long long k0 = (long long)q * " << CH << " + lane * 4;\n";
  if (mat_unit)
    e.o << "        if (k0 + 4 <= K) { const f4u w = " << e.ld(g.mat_group, "f4u", "Ar + k0") << "; xv[q][0] = w[0]; xv[q][1] = w[1]; xv[q][2] = w[2]; xv[q][3] = w[3]; }\n"
           "        else { for (int j = 0; j < 4; ++j) xv[q][j] = (k0 + j < K) ? Ar[k0 + j] : 0.0f; }\n";
  else
    e.o << "        for (int j = 0; j < 4; ++j) xv[q][j] = (k0 + j < K) ? Ar[(k0 + j) * ak] : 0.0f;\n";
  e.o << "      }\n#pragma unroll\n      for (int q = 0; q < " << KV << "; ++q)\n#pragma unroll\n        for (int j = 0; j < 4; ++j) acc = __builtin_fmaf(xv[q][j], wv[q][j], acc);\n";
  e.o << "    } else {\n      long long kb = 0;\n";
  if (mat_unit && vec_unit) {
    // long rows: four chunks per step, one dwordx4 of the row and of the vector per chunk and lane
    // (the vector comes from cache), four independent partial sums
    e.o << "      float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, a3 = 0.0f;\n";
    e.o << "      for (; kb + " << 4 * CH << " <= K; kb += " << 4 * CH << ") {\n        const long long k0 = kb + lane * 4;\n";
    for (int q = 0; q < 4; ++q)
      e.o << "        const f4u x" << q << " = " << e.ld(g.mat_group, "f4u", "Ar + k0 + " + std::to_string(q * CH)) << "; const f4u v" << q << " = *(const GM f4u*)(V + k0 + " << q * CH << ");\n";
    for (int q = 0; q < 4; ++q)
      e.o << "        for (int j = 0; j < 4; ++j) a" << q << " = __builtin_fmaf(x" << q << "[j], v" << q << "[j], a" << q << ");\n";
    e.o << "      }\n      acc = (a0 + a1) + (a2 + a3);\n";
  }
  e.o << "      for (; kb < K; kb += " << CH << ") {\n        const long long k0 = kb + lane * 4;\n";
  e.o << "        for (int j = 0; j < 4; ++j) if (k0 + j < K) acc = __builtin_fmaf(Ar[(k0 + j) * ak], V[(k0 + j) * vk], acc);\n      }\n    }\n";
  for (int m = LPR / 2; m > 0; m >>= 1) e.o << "    acc += gr_xor(acc, " << m << ");\n";
  e.o << "    if (lane == 0) {\n";
  gemv_epilogue(e, "row", "acc", "      ");
  e.o << "      out[row] = t" << g.results[0] << ";\n    }\n  }\n}\n";
}

// Second stage of the column-accumulate contraction: combines the slab partial vectors in a
// fixed order (deterministic; the two-kernel reduction of Section 3.2) and applies the epilogue.
void emit_colacc_combine(Em& e, const std::string& kname) {
  const GroupPlan& g = e.g;
  kernel_head(e, kname);
  e.o << "  const long long M = " << e.S(e.L.extra) << ", SLABS = " << e.S(e.L.extra + 3) << ";\n";
  e.o << "  const GM float* const ws = (const GM float*)" << e.slot(e.L.extra + 2) << ";\n";
  group_pointers(e, "  ", {g.mat_group, g.vec_group});
  // (few columns: four of a workgroup instead of sixteen, and a lane adds up its partial vectors in one round of loads; 384 and fewer, as the pieces
  // of a vector become short: 60000 x 333 21.0 -> 20.3 us, 378142 x 41 4.7 -> 4.0 of the kernel, but 120000 x 512 44.2 -> 44.7, 65536 x 2048 85.6 -> 90.5)
  e.o << "  const bool few = M <= " << kCombineFew << ";\n"
         "  const int tx = few ? threadIdx.x % 4 : threadIdx.x % 16, sg = few ? threadIdx.x / 4 : threadIdx.x / 16;\n"
         "  const long long m = (long long)blockIdx.x * (few ? 4 : 16) + tx;\n"
         "  __shared__ float sm[16][17];\n  float part = 0.0f, acc;\n"
         "  if (few) {\n"
         "    const int rows = (int)SLABS, of = (int)M, mc = m < M ? (int)m : 0;\n"
         "    for (int s = sg; s < rows; s += 512) {\n      float v[8];\n"
         "#pragma unroll\n      for (int u = 0; u < 8; ++u) v[u] = ws[(long long)(s + 64 * u < rows ? s + 64 * u : s) * of + mc];\n"
         "#pragma unroll\n      for (int u = 0; u < 8; ++u) part += s + 64 * u < rows ? v[u] : 0.0f;\n    }\n"
         "    for (int d = 4; d < 64; d *= 2) part += gr_xor(part, d);\n"
         "    if ((threadIdx.x & 63) < 4) sm[threadIdx.x >> 6][tx] = part;\n    __syncthreads();\n    acc = (sm[0][tx] + sm[1][tx]) + (sm[2][tx] + sm[3][tx]);\n"
         "  } else {\n"
         "    if (m < M) {\n      long long s = sg;\n"
         "      for (; s + 112 < SLABS; s += 128) {\n        float v[8];\n"
         "#pragma unroll\n        for (int u = 0; u < 8; ++u) v[u] = ws[(s + 16 * u) * M + m];\n"
         "#pragma unroll\n        for (int u = 0; u < 8; ++u) part += v[u];\n      }\n"
         "      for (; s < SLABS; s += 16) part += ws[s * M + m];\n    }\n"
         "    sm[sg][tx] = part;\n    __syncthreads();\n    acc = sm[0][tx];\n    for (int y = 1; y < 16; ++y) acc += sm[y][tx];\n  }\n";
  e.o << "  if (sg == 0 && m < M) {\n";
  gemv_epilogue(e, "m", "acc", "    ");
  e.o << "    ((GM float*)" << e.slot(e.L.out) << ")[m] = t" << g.results[0] << ";\n  }\n}\n";
}

void gen_gemv_colacc(Em& e) {
  const GroupPlan& g = e.g;
  const int BX = g.BX, BY = g.BY, UN = g.unroll;
  const AccessGroup& vg = g.groups[g.vec_group];
  const bool vec_unit = vg.coef[1] == 1;
  prelude(e);
  // stage 1: per-slab partial vectors
  kernel_head(e, kernel_name(g));
  e.o << "  const long long M = " << e.S(e.L.extra) << ", K = " << e.S(e.L.extra + 1) << ", SLABS = " << e.S(e.L.extra + 3) << ";\n";
  e.o << "  GM float* const ws = (GM float*)" << e.slot(e.L.extra + 2) << ";\n";
  group_pointers(e, "  ");
  e.o << "  const GM float* const A = q" << g.mat_group << "; const GM float* const V = q" << g.vec_group << ";\n";
  e.o << "  const long long ak = " << e.coef(g.mat_group, 1) << ", vk = " << (vec_unit ? std::string("1") : e.coef(g.vec_group, 1)) << ";\n";
  e.o << "  const int tx = threadIdx.x % " << BX << ", ty = threadIdx.x / " << BX << ";\n";
  e.o << "  const long long ncb = (M + " << BX * 4 - 1 << ") / " << BX * 4 << ";\n";
  e.o << "  const long long cb = blockIdx.x % ncb, slab = blockIdx.x / ncb;\n";
  e.o << "  const long long m0 = cb * " << BX * 4 << " + tx * 4;\n";
  e.o << "  const long long ks = (K + SLABS - 1) / SLABS, kbeg = slab * ks, kend = (kbeg + ks < K) ? kbeg + ks : K;\n";
  e.o << "  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};\n";
  e.o << "  if (m0 + 4 <= M) {\n"
         "    long long k = kbeg + ty;\n"
         "    for (; k + " << (UN - 1) * BY << " < kend; k += " << UN * BY << ") {\n"
         "      f4u x[" << UN << "]; float s[" << UN << "];\n"
         "#pragma unroll\n      for (int u = 0; u < " << UN << "; ++u) { x[u] = " << e.ld(g.mat_group, "f4u", "A + (k + u * " + std::to_string(BY) + ") * ak + m0") << "; s[u] = V[(k + u * " << BY << ") * vk]; }\n"
         "#pragma unroll\n      for (int u = 0; u < " << UN << "; ++u) { acc[0] = __builtin_fmaf(x[u][0], s[u], acc[0]); acc[1] = __builtin_fmaf(x[u][1], s[u], acc[1]); acc[2] = __builtin_fmaf(x[u][2], s[u], acc[2]); acc[3] = __builtin_fmaf(x[u][3], s[u], acc[3]); }\n"
         "    }\n"
         "    for (; k < kend; k += " << BY << ") { const f4u x = *(const GM f4u*)(A + k * ak + m0); const float s = V[k * vk];\n"
         "      acc[0] = __builtin_fmaf(x[0], s, acc[0]); acc[1] = __builtin_fmaf(x[1], s, acc[1]); acc[2] = __builtin_fmaf(x[2], s, acc[2]); acc[3] = __builtin_fmaf(x[3], s, acc[3]); }\n"
         "  } else {\n"
         "    for (long long k = kbeg + ty; k < kend; k += " << BY << ") { const float s = V[k * vk];\n"
         "      for (int j = 0; j < 4; ++j) if (m0 + j < M) acc[j] = __builtin_fmaf(A[k * ak + m0 + j], s, acc[j]); }\n"
         "  }\n";
  e.o << "  __shared__ float sm[" << BY << "][" << BX * 4 << "];\n";
  e.o << "  for (int j = 0; j < 4; ++j) sm[ty][tx * 4 + j] = acc[j];\n  __syncthreads();\n";
  e.o << "  if (ty == 0) {\n    for (int j = 0; j < 4; ++j) {\n      float t = sm[0][tx * 4 + j];\n      for (int y = 1; y < " << BY << "; ++y) t += sm[y][tx * 4 + j];\n"
         "      if (m0 + j < M) ws[slab * M + m0 + j] = t;\n    }\n  }\n}\n";
  emit_colacc_combine(e, kernel_name(g) + "_combine");
}

// Row-dot contraction, its epilogue, and the column-accumulate contraction that consumes the
// epilogue's result, in one pass over the matrix: a row stays in registers between
// z = X[i,:].w, r_i = epilogue(z) and g += X[i,:] * r_i.
// Bound by HBM where the waves, two per SIMD, have loads enough under way: one row at a time of 16 lanes each is 64 of them for 512 columns and
// eight for 41, and a load's latency is then paid once per row (378142 x 41: 50.9 us, 1.2 TB/s, 46 rows in turn at 1.1 us each).  With `unroll` rows
// at a time the loads of all of them come first; the end of a ragged row is one 16-byte load that starts earlier, instead of four under
// conditions that every row waited for as well; sums over the row's lanes are additions from neighbouring lanes' registers (of 16 lanes with the
// bits of the exchange through LDS); and lane u takes the epilogue of row u, which all lanes took for each row.
// (us of a logistic-regression step, before and after: 378142 x 41 53.8 / 15.7, 1000000 x 16 110 / 17.7, 300001 x 27 42.9 / 11.2, 249354 x 100 40.1 / 21.9,
// 526145 x 117 88.4 / 43.5, 1000000 x 64 98 / 46.5, 262144 x 192 39.9 / 35.9, 60000 x 333 26.3 / 20.3, 30000 x 700 24.8 / 19.5, 10000 x 2040 25.4 / 21.8)
void gen_gemv_pair(Em& e, Em& e2) {
  const GroupPlan& g = e.g;
  const int LPR = g.LPR, KV = g.KV, RPB = 256 / LPR, CH = LPR * 4, UN = g.unroll;
  const AccessGroup& mg = g.groups[g.mat_group];
  const AccessGroup& vg = g.groups[g.vec_group];
  (void)mg;
  const bool vec_unit = vg.coef[1] == 1;
  prelude(e);
  if (UN > 1) {
    // gr_from: the value of lane u of a row's lanes; gr_row_sum: the sum over them, in each of them
    e.o << "#define GR_DPP(v, c) __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), c, 0xf, 0xf, true))\n";
    if (LPR == 64) e.o << "#define gr_from(v, u) __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), u))\n";
    else if (LPR == 16) e.o << "#define gr_from(v, u) GR_DPP(v, 0x150 + u)\n";   // row_newbcast
    else e.o << "#define gr_from(v, u) __uint_as_float(__builtin_amdgcn_ds_swizzle(__float_as_uint(v), 0x18 | u << 5))\n";
    e.o << "static __device__ __forceinline__ float gr_row_sum(float v) {\n"
        << (LPR == 64 ? "  v += gr_xor(v, 32); v += gr_xor(v, 16);\n" : "")
        << (LPR == 8 ? "  v += GR_DPP(v, 0x141); v += GR_DPP(v, 0x4e); v += GR_DPP(v, 0xb1);\n"   // half mirror, quads turned by two and by one
                     : "  v += GR_DPP(v, 0x128); v += GR_DPP(v, 0x124); v += GR_DPP(v, 0x122); v += GR_DPP(v, 0x121);\n")   // turns by 8, 4, 2 and 1 lanes
        << "  return v;\n}\n";
  }
  kernel_head(e, "gr_gemv_pair");
  e.o << "  const long long M = " << e.S(e.L.extra) << ", K = " << e.S(e.L.extra + 1) << ", SLABS = " << e.S(e.L.extra + 3) << ";\n";
  e.o << "  GM float* const ws = (GM float*)" << e.slot(e.L.extra + 2) << ";\n";
  group_pointers(e, "  ");
  e.o << "  const GM float* const A = q" << g.mat_group << "; const GM float* const V = q" << g.vec_group << ";\n";
  e.o << "  const long long am = " << e.coef(g.mat_group, 0) << ", vk = " << (vec_unit ? std::string("1") : e.coef(g.vec_group, 1)) << ";\n";
  e.o << "  const int lane = threadIdx.x % " << LPR << ", rib = threadIdx.x / " << LPR << ";\n";
  e.o << "  GM float* const out = (GM float*)" << e.slot(e.L.out) << ";\n";
  e.o << "  const long long rs = ((M + SLABS - 1) / SLABS + " << RPB - 1 << ") / " << RPB << " * " << RPB << ";\n";
  e.o << "  const long long rbeg = (long long)blockIdx.x * rs, rend = (rbeg + rs < M) ? rbeg + rs : M;\n";
  if (UN == 1) {
    e.o << "  float wv[" << KV << "][4], acc[" << KV << "][4];\n";
    e.o << "#pragma unroll\n  for (int q = 0; q < " << KV << "; ++q) {\n    const long long k0 = (long long)q * " << CH << " + lane * 4;\n"
           "    for (int j = 0; j < 4; ++j) { wv[q][j] = (k0 + j < K) ? V[(k0 + j) * vk] : 0.0f; acc[q][j] = 0.0f; }\n  }\n";
    e.o << "  for (long long row = rbeg + rib; row < rend; row += " << RPB << ") {\n";
    e.o << "    const GM float* const Ar = A + row * am;\n    float xv[" << KV << "][4];\n";
    e.o << "#pragma unroll\n    for (int q = 0; q < " << KV << "; ++q) {\n      const long long k0 = (long long)q * " << CH << " + lane * 4;\n"
           "      if (k0 + 4 <= K) { const f4u w = " << e.ld(g.mat_group, "f4u", "Ar + k0") << "; xv[q][0] = w[0]; xv[q][1] = w[1]; xv[q][2] = w[2]; xv[q][3] = w[3]; }\n"
           "      else { for (int j = 0; j < 4; ++j) xv[q][j] = (k0 + j < K) ? Ar[k0 + j] : 0.0f; }\n    }\n";
    e.o << "    float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};\n"
           "#pragma unroll\n    for (int q = 0; q < " << KV << "; ++q)\n#pragma unroll\n      for (int j = 0; j < 4; ++j) z[j] = __builtin_fmaf(xv[q][j], wv[q][j], z[j]);\n"
           "    float zz = (z[0] + z[1]) + (z[2] + z[3]);\n";
    for (int m = LPR / 2; m > 0; m >>= 1) e.o << "    zz += gr_xor(zz, " << m << ");\n";
    gemv_epilogue(e, "row", "zz", "    ");
    e.o << "    const float rr = t" << g.results[0] << ";\n    if (lane == 0) out[row] = rr;\n";
    e.o << "#pragma unroll\n    for (int q = 0; q < " << KV << "; ++q)\n#pragma unroll\n      for (int j = 0; j < 4; ++j) acc[q][j] = __builtin_fmaf(xv[q][j], rr, acc[q][j]);\n  }\n";
  } else {
    // (the last chunk: a lane whose elements reach past the row's end reads the four before the end instead, and keeps those from its own first one on: zero in
    // both operands, as zero times an infinite weight is no number)
    e.o << "  const long long klast = " << (KV - 1) * CH << " + lane * 4, kb = klast + 4 <= K ? klast : K - 4;\n  const int skip = (int)(klast - kb < 4 ? klast - kb : 4);\n";
    e.o << "  float wv[" << KV << "][4], acc[" << KV << "][4];\n";
    e.o << "#pragma unroll\n  for (int q = 0; q < " << KV << "; ++q) {\n    const long long k0 = q == " << KV - 1 << " ? kb : (long long)q * " << CH << " + lane * 4;\n"
           "#pragma unroll\n    for (int j = 0; j < 4; ++j) { const float v = V[(k0 + j) * vk]; wv[q][j] = q < " << KV - 1 << " || skip <= j ? v : 0.0f; acc[q][j] = 0.0f; }\n  }\n";
    e.o << "  const int mine = lane < " << UN << " ? lane : 0;\n";
    e.o << "  const GM float* Ar = A + (rbeg + rib) * am;\n  long long row = rbeg + rib;\n";
    auto batch = [&](bool some, const char* ind) {
      const std::string I = ind;
      for (int u = 0; u < UN; ++u) {
        if (some && u) e.o << I << "const bool in" << u << " = row + " << u * RPB << " < rend;\n";
        e.o << I << "const GM float* const A" << u << " = " << (u == 0 ? "Ar" : some ? "in" + std::to_string(u) + " ? Ar + " + std::to_string(u * RPB) + " * am : Ar" : "Ar + " + std::to_string(u * RPB) + " * am") << ";\n";
        for (int q = 0; q < KV; ++q)
          e.o << I << "f4u x" << u << "_" << q << " = " << e.ld(g.mat_group, "f4u", "A" + std::to_string(u) + " + " + (q == KV - 1 ? std::string("kb") : std::to_string(q * CH) + " + lane * 4")) << ";\n";
      }
      e.o << I << "__builtin_amdgcn_sched_barrier(0);\n";
      for (int u = 0; u < UN; ++u) {
        const std::string x = "x" + std::to_string(u) + "_", z = "z" + std::to_string(u);
        e.o << I << "float " << z << ";\n" << I << "{\n";
        for (int j = 0; j < 4; ++j) e.o << I << "  " << x << KV - 1 << "[" << j << "] = skip <= " << j << " ? " << x << KV - 1 << "[" << j << "] : 0.0f;\n";
        for (int j = 0; j < 4; ++j) {
          e.o << I << "  float y" << j << " = " << x << "0[" << j << "] * wv[0][" << j << "];\n";
          for (int q = 1; q < KV; ++q) e.o << I << "  y" << j << " = __builtin_fmaf(" << x << q << "[" << j << "], wv[" << q << "][" << j << "], y" << j << ");\n";
        }
        e.o << I << "  " << z << " = gr_row_sum((y0 + y1) + (y2 + y3));\n" << I << "}\n";
      }
      // lane u of a row's lanes takes the epilogue of row u, for all of them
      e.o << I << "float zz = z0;\n";
      for (int u = 1; u < UN; ++u) e.o << I << "zz = mine == " << u << " ? z" << u << " : zz;\n";
      e.o << I << "const long long at = row + mine * " << RPB << ", ro = " << (some ? "at < rend ? at : row" : "at") << ";\n";
      gemv_epilogue(e, "ro", "zz", ind);
      e.o << I << "const float rr = t" << g.results[0] << ";\n" << I << "if (lane < " << UN << (some ? " && at < rend" : "") << ") out[at] = rr;\n";
      for (int u = 0; u < UN; ++u) {
        e.o << I << (some && u ? "if (in" + std::to_string(u) + ") " : std::string()) << "{\n" << I << "  const float r = gr_from(rr, " << u << ");\n";
        for (int q = 0; q < KV; ++q)
          for (int j = 0; j < 4; ++j) e.o << I << "  acc[" << q << "][" << j << "] = __builtin_fmaf(x" << u << "_" << q << "[" << j << "], r, acc[" << q << "][" << j << "]);\n";
        e.o << I << "}\n";
      }
    };
    e.o << "  for (; row + " << (UN - 1) * RPB << " < rend; row += " << UN * RPB << ", Ar += " << UN * RPB << " * am) {\n";
    batch(false, "    ");
    e.o << "  }\n  if (row < rend) {\n";
    batch(true, "    ");
    e.o << "  }\n";
  }
  // lanes with the same position in different row groups of a wave own the same columns
  e.o << "#pragma unroll\n  for (int q = 0; q < " << KV << "; ++q)\n#pragma unroll\n    for (int j = 0; j < 4; ++j) {\n";
  for (int m = LPR; m < 64; m <<= 1) e.o << "      acc[q][j] += gr_xor(acc[q][j], " << m << ");\n";
  e.o << "    }\n";
  e.o << "  __shared__ float sm[4][" << CH * KV << "];\n";
  if (UN == 1) e.o << "  if ((threadIdx.x & 63) < " << LPR << ") {\n#pragma unroll\n    for (int q = 0; q < " << KV << "; ++q)\n      for (int j = 0; j < 4; ++j) sm[threadIdx.x >> 6][q * " << CH << " + lane * 4 + j] = acc[q][j];\n  }\n";
  else e.o << "  if ((threadIdx.x & 63) < " << LPR << ") {\n#pragma unroll\n    for (int q = 0; q < " << KV << "; ++q)\n#pragma unroll\n      for (int j = 0; j < 4; ++j)\n"
              "        if (q < " << KV - 1 << " || skip <= j) sm[threadIdx.x >> 6][(q < " << KV - 1 << " ? q * " << CH << " + lane * 4 : (int)kb) + j] = acc[q][j];\n  }\n";
  e.o << "  __syncthreads();\n";
  e.o << "  for (int k = threadIdx.x; k < " << CH * KV << "; k += 256)\n    if (k < K) ws[(long long)blockIdx.x * K + k] = ((sm[0][k] + sm[1][k]) + sm[2][k]) + sm[3][k];\n}\n";
  // second stage with the second sub-graph's epilogue; its argument block follows the first one
  emit_colacc_combine(e2, "gr_gemv_pair_combine");
  e.o << e2.o.str();
}

// ---- GEMM (matrix cores) ----------------------------------------------------------

// The text fn writes to e.o, taken back out of the stream.
template <class F>
std::string captured(Em& e, F fn) {
  const std::string before = e.o.str();
  e.o.str("");
  fn();
  const std::string body = e.o.str();
  e.o.str(before);
  e.o.seekp(0, std::ios::end);
  return body;
}

// body once per combination of the loop variables, each a constant of its block.  Accumulators are register
// arrays, so every index into them has to be a constant or the array moves to scratch memory; the loops over them
// are unrolled here, in the text, because the compiler drops "#pragma unroll" once the unrolled size passes a
// threshold, which a long epilogue (tanh, erf, exp and log on 256 accumulators) does.
void emit_unrolled(std::ostream& o, const std::vector<std::pair<const char*, int>>& loops, const std::string& body, const char* ind) {
  std::vector<int> at(loops.size(), 0);
  for (;;) {
    o << ind << "{ constexpr int";
    for (size_t k = 0; k < loops.size(); ++k) o << (k ? ", " : " ") << loops[k].first << " = " << at[k];
    o << ";\n" << body << ind << "}\n";
    size_t k = loops.size();
    while (k > 0 && ++at[k - 1] == loops[k - 1].second) at[--k] = 0;
    if (k == 0) return;
  }
}

using EpiLoad = std::function<std::string(const Instr&, int)>;
void gemm_combine(Em& e, const EpiLoad& epi_load);

// Three bfloat16 pieces of a float32 value, x = h + m + l exactly, for the matrix products of gemm_big_body: each the rest rounded to
// nearest (eight bits, so that the last one is exact).  The matrix cores multiply bfloat16 pairs exactly and add them
// in float32 at sixteen times the float32 rate; eight of the nine products of pieces, all but l l, which is below 2^-34 of the
// product, take half of the time of float32 instructions.  Two things keep the sums at least as near 64 bits as those instructions'
// for any operands (results below 2^-122 apart, three units of the smallest denormal at most): the pieces lean to neither side (with a first piece that is cut off the small products of positive operands
// are all positive, and are lost where the sum has outgrown them: uniform values, K = 4096, 3.6e-6 for 8.4e-7), and the products below h h have
// sums of their own, because these matrix instructions do not round to nearest as float32 ones do (a single product per sum, 2048^3
// times a diagonal matrix: largest relative error of an element 6.0e-8 with float32 instructions, 1.2e-7 with all
// products in one sum, 2.9e-7 with six of them, 6.0e-8 so).
// What the pieces cannot hold is noticed as they are made, and the wave multiplies these and all further values of k with float32 instructions:
// of a value whose last piece would reach below the smallest denormal bfloat16 (a nonzero value below 2^-110 can
// be one) the low half of that piece, which is zero otherwise, is collected in `low`; of infinities, and of values whose products could make
// a sum of pieces overflow where the sum of the values does not, `big` keeps the largest magnitude (2^48 and more: gr_odd).
// (What is not a number is one in all of its products either way.)
// (us with 1e-35 at every 41st position of every 37th row / without such values / float32 instructions for all: 2048^3 147 / 120 / 134,
// 4096 x 512 x 784 40 / 34 / 42.)
// The splitting competes with the matrix instructions: about 6 vector instructions per value.  They overlap with other waves' matrix
// instructions; the two-term dot product instruction, which could take off a piece without unpacking it, does not (one wave with matrix
// instructions beside one with as many cycles of these: their sum; of the others a fifth more than the longer of the two).
void split_helpers(Em& e) {
  e.o << "typedef __bf16 gr_b2 __attribute__((ext_vector_type(2)));\n"
         "typedef __bf16 gr_b8 __attribute__((ext_vector_type(8)));\n"
         "typedef float gr_p2 __attribute__((ext_vector_type(2)));\n"
         "typedef unsigned gr_u4 __attribute__((ext_vector_type(4)));\n"
         "static __device__ __forceinline__ void gr_split2(float x0, float x1, unsigned& h, unsigned& m, unsigned& l, unsigned& low, float& big) {\n"
         "  h = __builtin_bit_cast(unsigned, __builtin_convertvector((gr_p2{x0, x1}), gr_b2));\n"
         "  const float r0 = x0 - __uint_as_float(h << 16), r1 = x1 - __uint_as_float(h & 0xffff0000u);\n"
         "  m = __builtin_bit_cast(unsigned, __builtin_convertvector((gr_p2{r0, r1}), gr_b2));\n"
         "  const unsigned l0 = __float_as_uint(r0 - __uint_as_float(m << 16)), l1 = __float_as_uint(r1 - __uint_as_float(m & 0xffff0000u));\n"
         "  l = __builtin_amdgcn_perm(l1, l0, 0x07060302u);\n"
         // (in place: left to the compiler, the collecting is put off and the pieces are kept in scratch memory for it)
         "  asm(\"v_or3_b32 %0, %0, %1, %2\" : \"+v\"(low) : \"v\"(l0), \"v\"(l1));\n"
         "  asm(\"v_max3_f32 %0, |%1|, |%2|, %0\" : \"+v\"(big) : \"v\"(x0), \"v\"(x1));\n}\n"
         "static __device__ __forceinline__ bool gr_odd(unsigned low, float big) { return __builtin_amdgcn_ballot_w64((low & 0xffffu) != 0u || big >= 0x1p48f) != 0ull; }\n";
}

// Matrix product of large operands, each contiguous along one of its dimensions (edge tiles load clamped rows and store only what exists; K no
// multiple of 16, and groups of four that are not whole, with two groups of waves only: GroupPlan::NP): one workgroup per tile of the
// result, tiles of 256 x 256 (four waves with a 128 x 128 quarter each as 4 x 4 matrix-core blocks, 256
// accumulator registers per lane) or 128 x 128 (one or two groups of four waves, 2 x 2 blocks per wave).
//   * Tiles of 16 values of k go from global memory straight into LDS (global_load_lds_dwordx4: lane L of a
//     wave deposits its 16 bytes at M0 + 16 L, whatever address it loaded them from), two steps ahead, into a
//     ring of three stages, so a step has one barrier, no staging registers and no LDS write instructions.
//   * A tile contiguous along k: rows of 16 floats; the four 16-byte chunks of row m sit at chunk position c ^ (m / 4 % 4),
//     which lets both the depositing wave (16 lanes = 4 rows x 4 chunks) and the reading one (16 lanes = 16
//     rows, one chunk) touch every bank once.  A lane reads the four k values of a chunk with one ds_read_b128
//     and feeds them to four matrix instructions: the instruction for element t of the chunks takes k = 4 h + t
//     (+ 8 in the second half of the step) in half-wave h instead of k = 2 s + h.  Both operands use the same
//     assignment, so every product is formed once; only the order of the additions differs.
//   * A tile contiguous along its other dimension: 16 rows of 256 floats with a pitch of 264 (rows 4 apart lie 32 banks apart).
//     Block j of a lane's four column blocks is column 4 r + j of the wave's 128 (r = lane % 32), so the four operands of a
//     k come with one ds_read_b128 and a lane's results are four neighbouring columns (16-byte stores).
//   * One group: float32 matrix instructions.  Per step and wave of the 256 x 256 tiles 128 of them, 16 LDS reads, 8 direct loads, one
//     barrier, each placed behind a fixed matrix instruction (scheduling barriers pin the order): with one wave per SIMD every
//     instruction between two matrix instructions delays the second one, which is what bounds this kernel
//     (measured on 4096^3, one variant each: staging through registers 137 TFLOP/s, direct loads 143, the
//     same with addresses precomputed and 16-byte reads of the right operand 151; a loop of nothing but
//     matrix instructions 154).
//   * Two groups: bfloat16 matrix instructions over three pieces of every value (split_helpers), which one wave per SIMD could not
//     both make and multiply in time.  A second set of sums fits here only (256 x 256 tiles have no registers for it; three workgroups of one
//     group per compute unit would be two: 3000 x 512 x 2048 72 us for 65 with float32 instructions).
//     (us, float32 instructions / pieces; relative error against 64 bits: 2048^3 132 / 119.5, 8.1e-7 / 1.9e-7; 4096 x 512 x 784 41.8 / 34.7,
//     4.1e-7 / 9.3e-8; 784 x 4096 x 512 44.4 / 38.8; 512 x 2848 x 2352 70 / 60.  With six products and one sum 101, 31.3, 35.4 and 52.)
//     Per wave and step 221 vector instructions, 32 of them conversions at half rate, 1010 cycles, and 32 matrix instructions, 1024. Bound by
//     both and by the clock that this load leaves (counters, 2048^3: of 200 thousand cycles the matrix cores work 66 %, the vector
//     units 69 %, both at once 40 %; 200 thousand cycles in 118 us are 1.7 GHz, where the float32 kernel runs at 2.3).
// The direct loads are written as assembly: the compiler's own form of them makes it wait for every outstanding
// LDS read before each use (it counts them as LDS traffic that may return out of order).  Their completion is
// tracked by hand: the wait before a step's barrier leaves only the loads of the newest tile in flight.
void gemm_big_body(Em& e, const EpiLoad& epi_load) {
  const GroupPlan& g = e.g;
  const int NB = g.BX / 64;          // matrix-core blocks per wave along each dimension: 4 (256 x 256 tiles) or 2 (128 x 128)
  const int T = 64 * NB, G = NB * NB, P = 2 * NB;   // tile edge, matrix instructions per group, direct loads per wave and step
  // An operand is either "k-contiguous" (kc: its tile is T rows of 16 k values, 16-byte chunks swizzled, a lane's
  // 16-byte read holds four k of one row and serves four matrix instructions) or "row-contiguous" (its tile is 16 k
  // rows of T values, a lane's read holds one k of NB neighbouring rows = its NB blocks).  Row-contiguous tiles of 256
  // values have a pitch of 264 floats (one row per load instruction); those of 128 values lie in pairs of rows (one
  // pair per load instruction) at a pitch of 272 per pair: rows four apart are 32 banks apart either way.
  struct Op { bool kc; const char* n; const char* ld; const char* org; const char* lim; int part; int size; };
  const bool akc = g.groups[g.mat_group].coef[1] == 1, bkc = g.groups[g.vec_group].coef[1] != 1;
  const int KC = T * 16, RC = NB == 4 ? 16 * 264 : 8 * 272;
  Op ops[2] = {{akc, "a", akc ? "am" : "ak", "bm0", "M", 0, akc ? KC : RC}, {bkc, "b", bkc ? "bn" : "bk", "bn0", "N", akc ? KC : RC, bkc ? KC : RC}};
  const int STAGE = ops[0].size + ops[1].size;   // floats
  auto rc_row = [&](int k) { return NB == 4 ? k * 264 : (k >> 1) * 272 + (k & 1) * 128; };   // offset of k row k of a row-contiguous tile (k without the half-wave's 4 h)
  const char* RV = NB == 4 ? "f4" : "gr_f2";      // what a lane reads of a row-contiguous tile per k
  std::ostream& o = e.o;
  const bool split = g.slabs > 1;
  const bool two = g.UC == 2;        // two groups of four waves
  o << "  __shared__ __attribute__((aligned(16))) float gr_lds[" << (two ? 6 : 3) * STAGE << "];\n"
       "  typedef __attribute__((address_space(3))) float lfloat;\n"
       "  typedef __attribute__((address_space(3))) f4 lf4;\n"
       "  typedef float gr_f2 __attribute__((ext_vector_type(2)));\n"
       "  typedef gr_f2 gr_f2u __attribute__((aligned(4)));\n"
       "  typedef __attribute__((address_space(3))) gr_f2 lgr_f2;\n"
       "  const int tid = threadIdx.x, lane = tid & 63, wave = " << (two ? "(tid >> 6) & 3" : "tid >> 6") << ", l32 = lane & 31, lh = lane >> 5;\n"
    << (two ? "  const int group = __builtin_amdgcn_readfirstlane(tid >> 8);\n" : "  const int group = 0;\n")
    << "  const int wm = (wave >> 1) * " << 32 * NB << ", wn = (wave & 1) * " << 32 * NB << ";\n"
       "  const long long tiles_n = (N + " << T - 1 << ") / " << T << ";\n";
  // split K (few output tiles, a long contraction): workgroup (tile, split) accumulates the steps of k in [kbeg, KE),
  // a whole number of steps and at least two by the planner's choice, and leaves its partial tile in a workspace
  if (split) o << "  const long long tiles = tiles_n * ((M + " << T - 1 << ") / " << T << "), tile = blockIdx.x % tiles, split = blockIdx.x / tiles;\n"
                  "  const long long kbeg = split * " << e.S(e.L.ocoef + 1) << ", KE = kbeg + " << e.S(e.L.ocoef + 1) << " < K ? kbeg + " << e.S(e.L.ocoef + 1) << " : K;\n";
  else o << "  const long long tile = blockIdx.x, kbeg = 0, KE = K;\n";
  // (ragged extents, see GroupPlan::NP: the last tile of a dimension that a row-contiguous operand has in groups of four starts T from its end
  // and overlaps the one before.  It stores only what lies from its place, bm1 and bn1, on: a wave that meets a value its pieces cannot hold sums
  // otherwise, and the two tiles' waves do not hold the same rows and columns, so the bits that both have stored would depend on which came last)
  const bool shift_m = g.NP & kGemmShiftM, shift_n = g.NP & kGemmShiftN;
  auto first = [&](const char* place, const char* lim, bool shifted) {
    const std::string end = std::string(lim) + " - " + std::to_string(T);
    return shifted ? "(" + std::string(place) + " < " + end + " ? " + place + " : " + end + ")" : std::string(place);
  };
  o << "  const long long bm1 = (tile / tiles_n) * " << T << ", bn1 = (tile % tiles_n) * " << T << ", bm0 = " << first("bm1", "M", shift_m) << ", bn0 = " << first("bn1", "N", shift_n) << ";\n"
       "  f16v acc[" << NB << "][" << NB << "];\n"
       "  for (int i = 0; i < " << NB << "; ++i) for (int j = 0; j < " << NB << "; ++j) for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.0f;\n"
       "  const unsigned wv = __builtin_amdgcn_readfirstlane(wave);\n"
       "  const lfloat* const ring = (const lfloat*)gr_lds + group * " << 3 * STAGE << ";\n"
       "  const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) void*)gr_lds + " << 12 * STAGE << "u * (unsigned)group;\n"
       "  const long long kfirst = kbeg + 16 * group;\n";
  for (const Op& x : ops) {
    const std::string n = x.n, w0 = x.n[0] == 'a' ? "wm" : "wn", X = x.n[0] == 'a' ? "A" : "B";
    // direct loads: a uniform base (advanced every step; made visibly uniform, the operands of the loads must be scalar
    // registers) plus a 32-bit byte offset per lane and piece
    o << "  unsigned " << n << "off[" << NB << "];\n#pragma unroll\n";
    if (x.kc)
      // (rows beyond the operand's edge read its last row: their results are never stored)
      o << "  for (int p = 0; p < " << NB << "; ++p) { const int m = 16 * (" << NB << " * wave + p) + lane / 4, c = (lane % 4) ^ ((m >> 2) & 3); const long long last = " << x.lim << " - 1 - " << x.org
        << "; " << n << "off[p] = 4u * (unsigned)((m < last ? m : last) * " << x.ld << " + 4 * c); }\n"
           "  const unsigned long long " << n << "64 = (unsigned long long)(" << X << " + " << x.org << " * " << x.ld << " + kfirst);\n"
           "  const unsigned long long " << n << "step = " << (two ? 128 : 64) << "ull;\n";
    else {
      // (groups of four beyond the operand's edge, whose extent is a multiple of four, read its last group)
      if (NB == 4) o << "  for (int p = 0; p < 4; ++p) { const long long last = " << x.lim << " - 4 - " << x.org << "; " << n << "off[p] = 4u * (unsigned)((4 * wave + p) * " << x.ld << " + (4 * lane < last ? 4 * lane : last)); }\n";
      else o << "  for (int p = 0; p < 2; ++p) { const long long last = " << x.lim << " - 4 - " << x.org << "; " << n << "off[p] = 4u * (unsigned)((2 * (2 * wave + p) + lane / 32) * " << x.ld << " + (4 * l32 < last ? 4 * l32 : last)); }\n";
      o << "  const unsigned long long " << n << "64 = (unsigned long long)(" << X << " + " << x.org << " + kfirst * " << x.ld << ");\n"
           "  const unsigned long long " << n << "step = " << (two ? 128 : 64) << "ull * (unsigned long long)__builtin_amdgcn_readfirstlane((int)" << x.ld << ");\n";
    }
    const int wave_bytes = x.kc ? 1024 * NB : (NB == 4 ? 4 * 264 * 4 : 4 * 272 * 2);
    o << "  unsigned long long " << n << "base = ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(" << n << "64 >> 32)) << 32) | (unsigned)__builtin_amdgcn_readfirstlane((int)" << n << "64);\n"
         "  unsigned " << n << "lds[3];\n#pragma unroll\n  for (int st = 0; st < 3; ++st) " << n << "lds[st] = lds0 + " << 4 * STAGE << "u * st + " << 4 * x.part << "u + " << wave_bytes << "u * wv;\n";
    // LDS read bases of this lane, per stage
    if (x.kc)
      o << "  const lfloat* " << n << "p[3][2];\n#pragma unroll\n  for (int st = 0; st < 3; ++st)\n#pragma unroll\n"
           "    for (int hf = 0; hf < 2; ++hf) " << n << "p[st][hf] = ring + st * " << STAGE << " + " << x.part << " + (" << w0 << " + l32) * 16 + 4 * ((2 * hf + lh) ^ ((l32 >> 2) & 3));\n"
           "";
    else
      o << "  const lfloat* " << n << "p[3];\n#pragma unroll\n  for (int st = 0; st < 3; ++st) " << n << "p[st] = ring + st * " << STAGE << " + " << x.part << " + " << rc_row(4) << " * lh + " << w0 << " + " << NB << " * l32;\n"
           "";
  }
  o << "  const long long nkt = (KE - kbeg) / 16;\n";
  // piece p (0 .. NB - 1: the left tile, NB .. 2 NB - 1: the right tile) of the tile at the bases into the stage in role st
  auto piece = [&](int st, int p, const char* ind) {
    const Op& x = ops[p / NB];
    const int imm = (x.kc ? 1024 : (NB == 4 ? 4 * 264 : 4 * 272)) * (p % NB);
    // The statement must not touch the scalar condition code: the compiler splits its own 64-bit additions (s_add_u32 ..
    // s_addc_u32) around it, so M0 is set with a move of a sum the compiler formed (an s_add_i32 here once corrupted the
    // carry of a base address: a memory fault).  The wait states cover what the compiler's hazard handling does not see
    // inside an asm statement: M0 written by a scalar instruction needs one before the load, a base address that a vector
    // instruction such as v_readfirstlane wrote needs five.
    o << ind << "asm volatile(\"s_mov_b32 m0, %2\\n\\ts_nop 4\\n\\tglobal_load_lds_dwordx4 %0, %1\" : : \"v\"("
      << x.n << "off[" << p % NB << "]), \"s\"(" << x.n << "base), \"s\"(" << x.n << "lds[" << st << "] + " << imm << "u) : \"memory\", \"m0\");\n";
  };
  // (Starting every workgroup's walk along k at a different step, so that workgroups running together read
  // different columns, was measured on 2048^3, whose rows of 8 KiB cost the 128 x 128-tile kernel a tenth against rows
  // padded by 64 bytes: no change, so the walk starts at zero everywhere.)
  const char* ADV = "abase += astep; bbase += bstep;\n";

  // the stages rotate through three roles (0: the tile of this step, 1: of the next one, 2: the target of this step's
  // loads): the addresses are exchanged after every step, a handful of register moves per step
  std::ostringstream rot;
  for (const Op& x : ops) {
    rot << "{ const unsigned t = " << x.n << "lds[0]; " << x.n << "lds[0] = " << x.n << "lds[1]; " << x.n << "lds[1] = " << x.n << "lds[2]; " << x.n << "lds[2] = t; }\n";
    if (x.kc) rot << "    { const lfloat* const t0 = " << x.n << "p[0][0]; const lfloat* const t1 = " << x.n << "p[0][1]; " << x.n << "p[0][0] = " << x.n << "p[1][0]; " << x.n << "p[0][1] = " << x.n << "p[1][1]; "
                  << x.n << "p[1][0] = " << x.n << "p[2][0]; " << x.n << "p[1][1] = " << x.n << "p[2][1]; " << x.n << "p[2][0] = t0; " << x.n << "p[2][1] = t1; }\n";
    else rot << "    { const lfloat* const t0 = " << x.n << "p[0]; " << x.n << "p[0] = " << x.n << "p[1]; " << x.n << "p[1] = " << x.n << "p[2]; " << x.n << "p[2] = t0; }\n";
    if (&x == &ops[0]) rot << "    ";
  }
  const std::string rot_text = rot.str();
  // What K leaves beyond its whole steps, fewer than 16 values, with float32 instructions from registers, in the second group, which has no more
  // steps than the first: loaded at once, zero beyond the end.
  auto rest = [&]() {
    if (!(g.NP & kGemmRestK)) return;
    o << "  { const long long krest = kbeg + 16 * nkt;\n  if (krest < KE && group == 1) {\n    float ar[8][" << NB << "], br[8][" << NB << "];\n";
    for (const Op& x : ops) {
      const std::string n = x.n, X = n == "a" ? "A" : "B", w0 = n == "a" ? "wm" : "wn";
      o << "#pragma unroll\n    for (int i = 0; i < " << NB << "; ++i) {\n"
           "      const long long at = " << x.org << " + " << w0 << " + " << (x.kc ? "32 * i + l32" : std::to_string(NB) + " * l32 + i") << ";\n"
           "      const GM float* const p = " << X << " + (at < " << x.lim << " ? at : " << x.lim << " - 1) * " << (n == "a" ? "am" : "bn") << ";\n"
           "#pragma unroll\n      for (int s = 0; s < 8; ++s) { const long long k = krest + 2 * s + lh; const float v = p[(k < KE ? k : krest) * " << (n == "a" ? "ak" : "bk") << "]; " << n << "r[s][i] = k < KE ? v : 0.0f; }\n    }\n";
    }
    o << "#pragma unroll\n    for (int s = 0; s < 8; ++s)\n#pragma unroll\n      for (int i = 0; i < " << NB << "; ++i)\n#pragma unroll\n        for (int j = 0; j < " << NB
      << "; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(ar[s][i], br[s][j], acc[i][j], 0, 0, 0);\n  } }\n";
  };
  if (two) {
    // Values t (t < 4) and 4 + t of a lane's eight are k = 4 h + t and 8 + 4 h + t in half-wave h, for both operands.
    // Block blk of an operand's tile in role 0.
    auto raw = [&](const Op& x, int blk, const char* ind) {
      const std::string n = x.n;
      for (int hf = 0; hf < 2; ++hf)
        o << ind << "{ const f4 w = *(const lf4*)(" << n << "p[0][" << hf << "] + " << blk * 512 << "); " << n << "r[" << blk << "][" << 4 * hf << "] = w[0]; " << n << "r[" << blk << "][" << 4 * hf + 1 << "] = w[1]; " << n << "r[" << blk << "][" << 4 * hf + 2 << "] = w[2]; " << n << "r[" << blk << "][" << 4 * hf + 3 << "] = w[3]; }\n";
    };
    auto raw_all = [&](const Op& x, const char* ind) {
      const std::string n = x.n;
      for (int blk = 0; x.kc && blk < NB; ++blk) raw(x, blk, ind);
      for (int v = 0; !x.kc && v < 8; ++v) {
        o << ind << "{ const " << RV << " w = *(const l" << RV << "*)(" << n << "p[0] + " << rc_row(8 * (v >> 2) + (v & 3)) << ");";
        for (int blk = 0; blk < NB; ++blk) o << ' ' << n << "r[" << blk << "][" << v << "] = w[" << blk << "];";
        o << " }\n";
      }
    };
    auto pieces_of = [&](const Op& x, int blk, int p, const char* ind) {
      const std::string n = x.n, to = n + "s[" + std::to_string(blk) + "]";
      o << ind << "{ unsigned h, m, l; gr_split2(" << n << "r[" << blk << "][" << 2 * p << "], " << n << "r[" << blk << "][" << 2 * p + 1 << "], h, m, l, low, big); " << to << "[0][" << p << "] = h; " << to << "[1][" << p << "] = m; " << to << "[2][" << p << "] = l; }\n";
    };
    static const int order[8][2] = {{2, 1}, {1, 2}, {2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};
    auto mfma = [&](int t, int i, int j, const char* ind) {
      const std::string to = std::string(t < 7 ? "tail[" : "acc[") + std::to_string(i) + "][" + std::to_string(j) + "]";
      o << ind << to << " = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(gr_b8, as[" << i << "][" << order[t][0] << "]), __builtin_bit_cast(gr_b8, bs[" << j << "][" << order[t][1] << "]), " << to << ", 0, 0, 0);\n";
    };
    const char* SB = "__builtin_amdgcn_sched_barrier(0);\n";
    for (const Op& x : ops) o << "  gr_u4 " << x.n << "s[" << NB << "][3];\n";
    const char* NONE_ODD = "unsigned low = 0u; float big = 0.0f;\n";
    // the tile in role 0 with float32 instructions, from LDS again (the values are not kept for it)
    auto exact = [&](const char* ind) {
      o << ind << "{ __atomic_signal_fence(__ATOMIC_SEQ_CST);\n" << ind << "float ar[" << NB << "][8], br[" << NB << "][8];\n";
      for (const Op& x : ops) raw_all(x, ind);
      for (int v = 0; v < 8; ++v) for (int i = 0; i < NB; ++i) for (int j = 0; j < NB; ++j)
        o << ind << "acc[" << i << "][" << j << "] = __builtin_amdgcn_mfma_f32_32x32x2f32(ar[" << i << "][" << v << "], br[" << j << "][" << v << "], acc[" << i << "][" << j << "], 0, 0, 0);\n";
      o << ind << "}\n";
    };
    // Group g of four waves takes every second step from step g on, its tiles in a ring of its own.  Vector and matrix instructions
    // of one wave hardly overlap, those of two waves of a SIMD do: between two barriers group 0 splits a tile and
    // multiplies it while group 1 multiplies the tile that it split before and splits the next (2048^3 with six products and
    // one sum, us: one group of four waves 133, two in step 120, these 108).
    o << "  f16v tail[2][2];\n  for (int i = 0; i < 2; ++i) for (int j = 0; j < 2; ++j) for (int q = 0; q < 16; ++q) tail[i][j][q] = 0.0f;\n";
    o << "  const int n0 = (int)((nkt + 1) / 2), mine = (int)((nkt + 1 - group) / 2);\n";
    auto fetch = [&](int role, const char* tile, const char* ind) {
      o << ind << "if (" << tile << " < mine) {\n";
      for (int p = 0; p < P; ++p) piece(role, p, ind);
      o << ind << ADV << ind << "}\n";
    };
    auto split_tile = [&](const char* ind) {
      o << ind << NONE_ODD;
      for (const Op& x : ops) {
        o << ind << "float " << x.n << "r[" << NB << "][8];\n";
        raw_all(x, ind);
      }
      for (const Op& x : ops) for (int blk = 0; blk < NB; ++blk) for (int p = 0; p < 4; ++p) pieces_of(x, blk, p, ind);
      o << ind << "if (gr_odd(low, big)) break;\n" << ind << SB;
    };
    auto products = [&](const char* ind) {
      for (int t = 0; t < 8; ++t) for (int i = 0; i < NB; ++i) for (int j = 0; j < NB; ++j) mfma(t, i, j, ind);
      o << ind << SB;
    };
    auto advance = [&](const char* ind) {   // the next tile has landed, all of this one's reads are done
      o << ind << "if (t + 2 < mine) __builtin_amdgcn_s_waitcnt(" << (0x0070 | P) << "); else __builtin_amdgcn_s_waitcnt(" << 0x0070 << ");\n" << ind << "__builtin_amdgcn_s_barrier();\n" << ind << rot_text;
    };
    // (each group, and a wave that meets a value the pieces cannot hold for what is left of its steps, has a loop of its own, with as many
    // barriers: where two ways to the same sums meet within a step, the compiler moves them about)
    fetch(0, "0", "  ");
    fetch(1, "1", "  ");
    o << "  if (mine > 1) __builtin_amdgcn_s_waitcnt(" << (0x0F70 | P) << "); else __builtin_amdgcn_s_waitcnt(" << 0x0F70 << ");\n  __builtin_amdgcn_s_barrier();\n  int t = 0;\n"
         "  if (group == 0) {\n    for (; t < mine; ++t) {\n";
    const char* ind = "      ";
    fetch(2, "t + 2", ind);
    split_tile(ind);
    products(ind);
    advance(ind);
    o << "    }\n    while (t < mine) {\n";
    exact(ind);
    advance(ind);
    o << ind << "++t;\n";
    fetch(2, "t + 2", ind);
    o << "    }\n  } else {\n";
    fetch(2, "2", "    ");
    o << "    for (; t < mine; ++t) {\n";
    split_tile(ind);
    advance(ind);
    fetch(2, "t + 3", ind);
    products(ind);
    o << "    }\n    while (t < mine) {\n";
    exact(ind);
    advance(ind);
    fetch(2, "t + 3", ind);
    o << ind << "++t;\n    }\n"
         "    if (mine < n0) __builtin_amdgcn_s_barrier();\n  }\n";
    rest();
    o << "#pragma unroll\n  for (int i = 0; i < 2; ++i)\n#pragma unroll\n    for (int j = 0; j < 2; ++j)\n#pragma unroll\n      for (int q = 0; q < 16; ++q) acc[i][j][q] += tail[i][j][q];\n";
    // the groups add up their sums: each takes one row of blocks
    o << "  f16v own[2];\n"
         "  { f4* const area = (f4*)gr_lds + (wave * 8) * 64 + lane;   // 32 KiB per group: what it leaves to the other one\n"
         "#pragma unroll\n    for (int j = 0; j < 2; ++j)\n#pragma unroll\n      for (int q = 0; q < 16; ++q) { const float a = acc[0][j][q], b = acc[1][j][q]; own[j][q] = group ? b : a; acc[0][j][q] = group ? a : b; }\n"
         "#pragma unroll\n    for (int j = 0; j < 2; ++j)\n#pragma unroll\n      for (int q = 0; q < 4; ++q) area[group * 2048 + (j * 4 + q) * 64] = f4{acc[0][j][4 * q], acc[0][j][4 * q + 1], acc[0][j][4 * q + 2], acc[0][j][4 * q + 3]};\n"
         "    __syncthreads();\n"
         "#pragma unroll\n    for (int j = 0; j < 2; ++j)\n#pragma unroll\n      for (int q = 0; q < 4; ++q) { const f4 v = area[(1 - group) * 2048 + (j * 4 + q) * 64]; own[j][4 * q] += v[0]; own[j][4 * q + 1] += v[1]; own[j][4 * q + 2] += v[2]; own[j][4 * q + 3] += v[3]; }\n"
         "  }\n";
  } else {
    const char* SB = "__builtin_amdgcn_sched_barrier(0);\n";
    for (const Op& x : ops)
      if (x.kc) o << "  f4 " << x.n << "F[2][" << NB << "];\n";
      else o << "  " << RV << " " << x.n << "F[2];\n";
    // operand of a matrix instruction (group s of the step, block blk) and the LDS reads that provide it
    auto val = [&](const Op& x, int s, int blk) {
      std::ostringstream v;
      if (x.kc) v << x.n << "F[" << (s >> 2) << "][" << blk << "][" << (s & 3) << "]";
      else v << x.n << "F[" << (s & 1) << "][" << blk << "]";
      return v.str();
    };
    auto read_kc = [&](const Op& x, int st, int hf, int blk, const char* ind) {
      o << ind << x.n << "F[" << hf << "][" << blk << "] = *(const lf4*)(" << x.n << "p[" << st << "][" << hf << "] + " << blk * 512 << ");\n";
    };
    auto read_rc = [&](const Op& x, int st, int s, const char* ind) {
      o << ind << x.n << "F[" << (s & 1) << "] = *(const l" << RV << "*)(" << x.n << "p[" << st << "] + " << rc_row(8 * (s >> 2) + (s & 3)) << ");\n";
    };
    // One step.  Role 0 is the stage that holds the current tile; the tile two steps on goes to the stage in role 2 if more2;
    // the first operands of the next step are read (from role 1) behind the barrier if more1.  Every load and LDS read
    // sits behind a fixed matrix instruction of a fixed group.
    auto step = [&](bool more2, bool more1, const char* ind) {
      for (int s = 0; s < 8; ++s) {
        if (s == 7)
          // the next tile has landed (all but the newest P loads are complete) and this wave's reads of the current one are done
          o << ind << "__builtin_amdgcn_s_waitcnt(" << (more2 ? 0x0070 | P : 0x0070) << ");\n" << ind << "__builtin_amdgcn_s_barrier();\n";
        for (int q = 0; q < G; ++q) {
          const int i = q / NB, j = q % NB;
          o << ind << SB << ind << "acc[" << i << "][" << j << "] = __builtin_amdgcn_mfma_f32_32x32x2f32(" << val(ops[0], s, i) << ", " << val(ops[1], s, j)
            << ", acc[" << i << "][" << j << "], 0, 0, 0);\n" << ind << SB;
          if (more2 && q == 1 && s < P && s < 7) piece(2, s, ind);
          if (more2 && NB == 4 && s == 6 && q == 9) piece(2, 7, ind);
          if (more2 && s == (NB == 4 ? 6 : 3) && q == (NB == 4 ? 9 : 1)) o << ind << ADV;
          for (int k = 0; k < 2; ++k) {
            const Op& x = ops[k];
            if (x.kc) {
              // second half of the step: behind the last NB matrix instructions of group 1 (left) / 2 (right);
              // first half of the next step: behind the first 2 NB of group 7
              if (s == 1 + k && q >= G - NB) read_kc(x, 0, 1, q - (G - NB), ind);
              if (s == 7 && more1 && q >= NB * k && q < NB + NB * k) read_kc(x, 1, 0, q - NB * k, ind);
            } else {
              if (s < 7 && q == NB + k) read_rc(x, 0, s + 1, ind);
              if (s == 7 && more1 && q == NB + k) read_rc(x, 1, 0, ind);
            }
          }
        }
      }
    };
    // prologue: tiles 0 and 1 (K >= 32)
    for (int t = 0; t < 2; ++t) {
      for (int p = 0; p < P; ++p) piece(t, p, "  ");
      o << "  " << ADV;
    }
    o << "  __builtin_amdgcn_s_waitcnt(" << (0x0F70 | P) << ");\n  __builtin_amdgcn_s_barrier();\n";
    for (const Op& x : ops) {
      if (x.kc) for (int blk = 0; blk < NB; ++blk) read_kc(x, 0, 0, blk, "  ");
      else read_rc(x, 0, 0, "  ");
    }
    o << "  long long kt = 0;\n"
         "  for (; kt + 2 < nkt; ++kt) {\n";
    step(true, true, "    ");
    o << "    " << rot_text << "  }\n"
         "  // the last two steps load nothing\n";
    step(false, true, "  ");
    o << "  " << rot_text;
    step(false, false, "  ");
  }
  // epilogue on the accumulators: element q of a block is its row rr = 8 (q / 4) + 4 (lane / 32) + q % 4 and column lane % 32;
  // block i of a k-contiguous left operand holds rows wm + 32 i + rr, of a row-contiguous one rows wm + NB rr + i; block j
  // of a row-contiguous right operand holds column wn + NB (lane % 32) + j (a lane's NB results are neighbours: one
  // vector store), of a k-contiguous one column wn + 32 j + lane % 32.
  // Results beyond the edges of the matrix are computed like the others, from operands read at the clamped position,
  // and not stored (no branch around the epilogue: sixty-four guarded copies of a large one made the register
  // allocator spill).
  if (split) o << "  GM float* const out = (GM float*)" << e.slot(e.L.ocoef) << " + split * M * N;\n";   // the partial tile; gr_gemm_combine applies the epilogue
  else o << "  GM float* const out = (GM float*)" << e.slot(e.L.out) << ";\n";
  const std::string body = captured(e, [&] {
    o << "      const int rr = 8 * (q / 4) + 4 * lh + (q % 4);\n"
         "      const long long row_at = bm0 + wm + " << (two ? (ops[0].kc ? "32 * group + rr" : "2 * rr + group") : (ops[0].kc ? "32 * i + rr" : std::to_string(NB) + " * rr + i")) << ", row = row_at < M ? row_at : M - 1;\n"
         "      " << RV << " ov;\n"
         "#pragma unroll\n      for (int j = 0; j < " << NB << "; ++j) {\n"
         "        const long long col_at = bn0 + wn + " << (ops[1].kc ? "32 * j + l32" : std::to_string(NB) + " * l32 + j") << ", col = col_at < N ? col_at : N - 1;\n"
         "        const float cacc = " << (two ? "own[j][q]" : "acc[i][j][q]") << ";\n";
    std::string res = "cacc";
    if (!split) { emit_scalar_program(e, g.prog, g.results, epi_load, "cacc", "t", "        "); res = "t" + std::to_string(g.results[0]); }
    const std::string in_rows = std::string(shift_m ? "row_at >= bm1 && " : "") + "row_at < M";
    if (ops[1].kc) o << "        if (" << in_rows << " && col_at < N) out[row * N + col] = " << res << ";\n      }\n      (void)ov;\n";
    else {
      o << "        ov[j] = " << res << ";\n      }\n"
           "      const long long at = bn0 + wn + " << NB << " * l32;\n"
           "      if (" << in_rows << " && at < N" << (shift_n ? " && at >= bn1" : "") << ") *(GM " << RV << "u*)(out + row * N + at) = ov;\n";
      if (shift_n) o << "      else if (" << in_rows << " && at + 1 == bn1) out[row * N + bn1] = ov[1];\n";   // (NB = 2: the second of a pair)
    }
  });
  if (two) emit_unrolled(o, {{"q", 16}}, body, "    ");
  else emit_unrolled(o, {{"i", NB}, {"q", 16}}, body, "    ");
  o << "}\n";
}


// Products that do not fill rounds of large tiles, of any extents (each operand contiguous along one of its two
// dimensions, extents of four or more): tiles of TM x TN = 64 x 64, 128 x 32 or 32 x 128, a 32 x 32 block per wave,
// several workgroups per compute unit.  Small products are bound by the latency of their loads and by compute units
// without a tile, ragged ones by guarded loads: here K advances 32 at a time, the loads run three steps ahead in
// registers, and no load is guarded.  The last tile of a dimension starts T from its end and overlaps the one before it
// with the same values; where an operand is narrower than a tile, rows (or groups of four) beyond its end are clamped
// to its last ones, and results for them are not stored.  The last step of K is shifted into place and padded with
// zeros on its way into LDS.
// LDS: an operand contiguous along k lies as [other][k] at a pitch of 36, read four k at a time; one contiguous along
// its other dimension as [k][other] at a pitch of T + 8, read one k at a time; both without bank conflicts.  Half-wave
// h takes k = 8 g + 4 h + t in matrix instruction t of group g, for both operands.  Loads, LDS reads and LDS writes of a
// step are placed one behind each matrix instruction (scheduling barriers): waves that do them in a phase of their own
// leave the matrix cores idle together, however many there are.
void gemm_tile_body(Em& e, const EpiLoad& epi_load) {
  const GroupPlan& g = e.g;
  std::ostream& o = e.o;
  const int TT[2] = {g.BY, g.BX}, S = 3, KS = 32, G = KS / 8;   // S: steps in flight
  const int groups[2] = {g.mat_group, g.vec_group};
  bool kc[2];
  int nv[2], pitch[2], rows[2];
  for (int x = 0; x < 2; ++x) {
    const AccessGroup& ag = g.groups[groups[x]];
    kc[x] = ag.coef[x == 0 ? 1 : 0] == 1;
    nv[x] = TT[x] * KS / 4 / 256;
    pitch[x] = kc[x] ? KS + 4 : TT[x] + 8;
    rows[x] = kc[x] ? TT[x] : KS;
  }
  const char* nm[2] = {"A", "B"};
  const char* ext[2] = {"M", "N"};
  const char* org[2] = {"bm0", "bn0"};
  for (int x = 0; x < 2; ++x) o << "  __shared__ __attribute__((aligned(16))) float S" << nm[x] << "[2][" << rows[x] << "][" << pitch[x] << "];\n";
  o << "  const unsigned tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, lh = lane >> 5;\n"
       "  const unsigned wm = " << (g.BY == 64 ? "(wave >> 1) * 32" : (g.BY == 128 ? "wave * 32" : "0")) << ", wn = " << (g.BX == 64 ? "(wave & 1) * 32" : (g.BX == 128 ? "wave * 32" : "0")) << ";\n"
       "  const long long NSPLIT = " << e.S(e.L.extra + 3) << ", KCH = " << e.S(e.L.ocoef + 1) << ";\n"
       "  const unsigned tiles_n = (unsigned)((N + " << TT[1] - 1 << ") / " << TT[1] << "), tiles = tiles_n * (unsigned)((M + " << TT[0] - 1 << ") / " << TT[0] << "), total = tiles * (unsigned)NSPLIT;\n"
       // (neighbouring tiles share operand rows: they go to the same XCD, workgroups are dealt round-robin over the 8)
       "  const unsigned per = (total + 7) / 8, job = (blockIdx.x % 8) * per + blockIdx.x / 8;\n"
       "  if (blockIdx.x / 8 >= per || job >= total) return;\n"
       "  const unsigned split = job / tiles, tile = job % tiles;\n"
       "  const long long bm1 = (long long)(tile / tiles_n) * " << TT[0] << ", bn1 = (long long)(tile % tiles_n) * " << TT[1] << ";\n"
       "  const long long bm0 = bm1 + " << TT[0] << " <= M || M < " << TT[0] << " ? bm1 : M - " << TT[0] << ", bn0 = bn1 + " << TT[1] << " <= N || N < " << TT[1] << " ? bn1 : N - " << TT[1] << ";\n"
       "  const long long kbeg = split * KCH, KE = (kbeg + KCH < K) ? kbeg + KCH : K;\n"
       "  const int kn = KE > kbeg ? (int)(KE - kbeg) : 0, nkt = (kn + " << KS - 1 << ") / " << KS << ", nfull = kn / " << KS << ", klast = (int)(KE - kbeg);\n";
  for (int x = 0; x < 2; ++x) {
    o << "  f4 r" << nm[x] << "[" << S << "][" << nv[x] << "];\n";
    if (!kc[x]) o << "  const unsigned s" << nm[x] << " = (unsigned)" << (x == 0 ? "ak" : "bk") << ";;\n";
    for (int v = 0; v < nv[x]; ++v) {
      const std::string id = std::string(nm[x]) + std::to_string(v);
      o << "  const unsigned i" << id << " = tid + " << 256 * v << ";\n";
      if (kc[x]) {
        o << "  const unsigned k" << id << " = i" << id << " % " << KS / 4 << " * 4, o" << id << " = i" << id << " / " << KS / 4 << ";\n"
             "  const GM float* const p" << id << " = " << nm[x] << " + (" << org[x] << " + o" << id << " < " << ext[x] << " ? " << org[x] << " + o" << id << " : " << ext[x] << " - 1) * " << (x == 0 ? "am" : "bn") << " + kbeg;\n";
      } else {
        o << "  const unsigned k" << id << " = i" << id << " / " << TT[x] / 4 << ", h" << id << " = i" << id << " % " << TT[x] / 4 << " * 4;\n"
             "  const unsigned o" << id << " = " << org[x] << " + h" << id << " + 4 <= " << ext[x] << " ? h" << id << " : (unsigned)(" << ext[x] << " - 4 - " << org[x] << ");\n"
             "  const GM float* const p" << id << " = " << nm[x] << " + " << org[x] << " + o" << id << " + kbeg * " << (x == 0 ? "ak" : "bk") << ";\n";
      }
    }
  }
  // (an operand narrower than its tile has origin 0: a clamped group of four starts at ext - 4 >= 0)
  auto fetch = [&](int x, int v, int set, const std::string& kt) {
    const std::string id = std::string(nm[x]) + std::to_string(v), at = "((" + kt + ") * " + std::to_string(KS) + " + (int)k" + id + ")", to = std::string("r") + nm[x] + "[" + std::to_string(set) + "][" + std::to_string(v) + "]";
    if (kc[x]) o << "        { const int k = " << at << " + 4 <= kn ? " << at << " : klast - 4; " << to << " = *(const GM f4u*)(p" << id << " + k); }\n";
    else o << "        { const int k = " << at << " < kn ? " << at << " : klast - 1; " << to << " = *(const GM f4u*)(p" << id << " + (unsigned long long)(unsigned)k * s" << nm[x] << "); }\n";
  };
  auto stash = [&](int x, int v, int set, const std::string& kt, bool tail) {
    const std::string id = std::string(nm[x]) + std::to_string(v);
    o << "        { f4 w = r" << nm[x] << "[" << set << "][" << v << "]; const int kt1 = " << kt << ", nb = kt1 & 1;\n";
    if (kc[x]) {
      if (tail)
        o << "          { const int k = kt1 * " << KS << " + (int)k" << id << ", sh = k + 4 <= kn ? 0 : k + 4 - kn; f4 z;\n"
             "            z[0] = sh == 0 ? w[0] : sh == 1 ? w[1] : sh == 2 ? w[2] : w[3]; z[1] = sh == 0 ? w[1] : sh == 1 ? w[2] : w[3]; z[2] = sh == 0 ? w[2] : w[3]; z[3] = w[3];\n"
             "            w[0] = k < kn ? z[0] : 0.0f; w[1] = k + 1 < kn ? z[1] : 0.0f; w[2] = k + 2 < kn ? z[2] : 0.0f; w[3] = k + 3 < kn ? z[3] : 0.0f; }\n";
      o << "          *(f4*)&S" << nm[x] << "[nb][o" << id << "][k" << id << "] = w; }\n";
    } else {
      if (tail) o << "          if (kt1 * " << KS << " + (int)k" << id << " >= kn) w = f4{0.0f, 0.0f, 0.0f, 0.0f};\n";
      // (a clamped group of an operand that is no multiple of four wide is not aligned in LDS)
      if ((g.NP - 1) >> x & 1) o << "          for (int j = 0; j < 4; ++j) S" << nm[x] << "[nb][k" << id << "][o" << id << " + j] = w[j]; }\n";
      else o << "          *(f4*)&S" << nm[x] << "[nb][k" << id << "][o" << id << "] = w; }\n";
    }
  };
  auto read = [&](int x, int gr) {
    const std::string to = std::string(x == 0 ? "a" : "b") + std::to_string(gr), w0 = x == 0 ? "wm" : "wn";
    if (kc[x]) o << "        " << to << " = *(const f4*)&S" << nm[x] << "[buf][" << w0 << " + l32][" << 8 * gr << " + 4 * lh];\n";
    else for (int t = 0; t < 4; ++t) o << "        " << to << "[" << t << "] = S" << nm[x] << "[buf][" << 8 * gr + t << " + 4 * lh][" << w0 << " + l32];\n";
  };
  // one step of K: tile kt (in LDS), loads of tile kt + S into register set `set` (or none), tile kt + 1 from its set to LDS
  auto step = [&](const std::string& kt, int set, bool loads, int stash_mode /* 0 none, 1 whole tile, 2 perhaps the last one */) {
    std::vector<std::function<void()>> piece;
    if (loads) for (int x = 0; x < 2; ++x) for (int v = 0; v < nv[x]; ++v) piece.push_back([&, x, v] { fetch(x, v, set, kt + " + " + std::to_string(S)); });
    const size_t nl = piece.size();
    for (int gr = 2; gr < G; ++gr) for (int x = 0; x < 2; ++x) piece.push_back([&, x, gr] { read(x, gr); });
    if (stash_mode == 1) for (int x = 0; x < 2; ++x) for (int v = 0; v < nv[x]; ++v) piece.push_back([&, x, v] { stash(x, v, (set + 1) % S, kt + " + 1", false); });
    o << "      {\n        const int buf = (" << kt << ") & 1;\n        f4 ";
    for (int gr = 0; gr < G; ++gr) o << "a" << gr << ", b" << gr << (gr + 1 < G ? ", " : ";\n");
    for (int gr = 0; gr < 2; ++gr) for (int x = 0; x < 2; ++x) read(x, gr);
    o << "        __builtin_amdgcn_sched_barrier(0);\n";
    size_t at = 0;
    for (int m = 0; m < 4 * G; ++m) {
      const int gr = m / 4, t = m % 4;
      const char* ac = m % 2 ? "acc2" : "acc";   // (two sets of accumulators: half as many additions in a row)
      o << "        " << ac << " = __builtin_amdgcn_mfma_f32_32x32x2f32(a" << gr << "[" << t << "], b" << gr << "[" << t << "], " << ac << ", 0, 0, 0);\n        __builtin_amdgcn_sched_barrier(0);\n";
      // (the operands of group 2 are read behind the first four instructions at the latest, those of group 3 behind eight;
      // the first LDS write waits for its load as long as it can)
      size_t upto = at;
      if (m < 6) upto = std::max(at, std::min(piece.size(), (size_t)(m + 1) * (nl + 4) / 6));
      else if (stash_mode == 1) upto = std::min(piece.size(), nl + 4 + (size_t)std::max(0, m - 5));
      else upto = piece.size();
      if (upto > at) {
        for (; at < upto; ++at) piece[at]();
        o << "        __builtin_amdgcn_sched_barrier(0);\n";
      }
    }
    for (; at < piece.size(); ++at) piece[at]();
    if (stash_mode == 2) {
      o << "        if (" << kt << " + 1 < nkt) {\n";
      for (int x = 0; x < 2; ++x) for (int v = 0; v < nv[x]; ++v) stash(x, v, (set + 1) % S, kt + " + 1", true);
      o << "        }\n";
    }
    o << "        __syncthreads();\n      }\n";
  };
  o << "  f16v acc, acc2;\n  for (int q = 0; q < 16; ++q) acc[q] = acc2[q] = 0.0f;\n  if (nkt > 0) {\n";
  for (int u = 0; u < S; ++u) for (int x = 0; x < 2; ++x) for (int v = 0; v < nv[x]; ++v) fetch(x, v, u, std::to_string(u));
  for (int x = 0; x < 2; ++x) for (int v = 0; v < nv[x]; ++v) stash(x, v, 0, "0", true);
  // (no condition around the loads of the main loop: the compiler would wait for them where the paths meet)
  o << "    __syncthreads();\n    int kt = 0;\n    for (; kt + " << S << " < nfull; kt += " << S << ") {\n";
  for (int u = 0; u < S; ++u) step("kt + " + std::to_string(u), u, true, 1);
  // one to S + 1 tiles are left (the last of them perhaps partial), all but the last of S + 1 in flight
  o << "    }\n";
  for (int u = 0; u <= S; ++u) {
    if (u) o << "    if (kt + " << u << " < nkt)\n";
    step("kt + " + std::to_string(u), u % S, u == 0, u < S ? 2 : 0);
  }
  o << "  }\n  acc += acc2;\n  GM float* const out = (GM float*)" << e.slot(e.L.out) << ";\n"
       "  if (NSPLIT > 1) {\n    GM float* const ws = (GM float*)" << e.slot(e.L.ocoef) << " + split * M * N;\n"
       "#pragma unroll\n    for (int q = 0; q < 16; ++q) {\n"
       "      const long long row = bm0 + wm + 8 * (q / 4) + 4 * lh + (q % 4), col = bn0 + wn + l32;\n"
       "      if (row < M && col < N) ws[row * N + col] = acc[q];\n    }\n    return;\n  }\n";
  const std::string body = captured(e, [&] {
    o << "#pragma unroll\n      for (int ql = 0; ql < 4; ++ql) {\n"
         "      const int q = 4 * qh + ql;\n"
         "      const long long row = bm0 + wm + 8 * qh + 4 * lh + ql, col = bn0 + wn + l32;\n"
         "      if (row < M && col < N) {\n        const float cacc = acc[q];\n";
    emit_scalar_program(e, g.prog, g.results, epi_load, "cacc", "t", "        ");
    o << "        out[row * N + col] = t" << g.results[0] << ";\n      }\n      }\n";
  });
  emit_unrolled(o, {{"qh", 4}}, body, "    ");
  o << "}\n";
}

// Short sums, and small results with any sum: every wave takes a block of 32 x 32 and loads its operands in the order in which the
// matrix instructions want them, straight into registers; nothing goes through LDS and no wave waits for another one before the end.
// UC = 1: the waves of a workgroup lie side by side (BY x BX).  Bound by stores and by the latency of a wave's few loads, which the
// other waves of its SIMD hide: many small waves, where tiles of 64 x 64 and 128 x 128 leave one or two workgroups to a compute unit that load,
// multiply and store one after the other.
// UC = 8: a workgroup is one block, whose values of k eight waves divide among themselves; they meet in LDS, and every lane finishes two
// results.  Bound by latency: as many compute units as there are blocks work on a result that is a few tiles of 64 x 64, and a chain of
// matrix instructions is an eighth as long.
// (operands in fragment order come at about 20 bytes per cycle and compute unit where they are contiguous along k, see gemm_tile_body for long sums)
void gemm_block_body(Em& e, const EpiLoad& epi_load) {
  const GroupPlan& g = e.g;
  std::ostream& o = e.o;
  const int KW = g.UC, WN = KW > 1 ? 1 : g.BX / 32, NK = 16;   // NK: values of k per step of the loop
  const bool kc[2] = {g.groups[g.mat_group].coef[1] == 1, g.groups[g.vec_group].coef[0] == 1};
  const char* nm[2] = {"A", "B"};
  o << "  const unsigned lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, lh = lane >> 5;\n"
       "  const long long NSPLIT = " << e.S(e.L.extra + 3) << ", KCH = " << e.S(e.L.ocoef + 1) << ";\n"
       "  const unsigned tiles_n = (unsigned)((N + " << g.BX - 1 << ") / " << g.BX << "), tiles = tiles_n * (unsigned)((M + " << g.BY - 1 << ") / " << g.BY << "), total = tiles * (unsigned)NSPLIT;\n"
       // (neighbouring tiles share operand rows: they go to the same XCD, workgroups are dealt round-robin over the 8)
       "  const unsigned per = (total + 7) / 8, job = (blockIdx.x % 8) * per + blockIdx.x / 8;\n"
       "  if (blockIdx.x / 8 >= per || job >= total) return;\n"
       "  const unsigned split = job / tiles, tile = job % tiles;\n"
       "  const long long m0 = (long long)(tile / tiles_n) * " << g.BY << (KW > 1 ? "" : " + wave / " + std::to_string(WN) + " * 32") << ", n0 = (long long)(tile % tiles_n) * " << g.BX << (KW > 1 ? "" : " + wave % " + std::to_string(WN) + " * 32") << ";\n";
  if (KW == 1) o << "  if (m0 >= M || n0 >= N) return;\n";
  o << "  const long long k0 = split * KCH, k1 = k0 + KCH < K ? k0 + KCH : K;\n";
  // (a wave's share of k: whole groups of eight)
  if (KW > 1) o << "  const long long share = ((k1 > k0 ? k1 - k0 : 0) + " << 8 * KW - 1 << ") / " << 8 * KW << " * 8, kb = k0 + wave * share, ke = kb + share < k1 ? kb + share : k1;\n";
  else o << "  const long long kb = k0, ke = k1;\n";
  o << "  const GM float* pA = A + (m0 + l32 < M ? m0 + l32 : M - 1) * am + (kb + 4 * lh) * ak;\n"
       "  const GM float* pB = B + (n0 + l32 < N ? n0 + l32 : N - 1) * bn + (kb + 4 * lh) * bk;\n"
       "  f16v acc, acc2;\n#pragma unroll\n  for (int q = 0; q < 16; ++q) acc[q] = acc2[q] = 0.0f;\n"
       "  const int n = ke > kb ? (int)(ke - kb) : 0;\n  int k = 0;\n";
  auto whole = [&](const char* to, int groups) {   // groups of eight values of k, all there
    for (int x = 0; x < 2; ++x)
      for (int gr = 0; gr < groups; ++gr) {
        const std::string v = std::string(to) + nm[x] + std::to_string(gr), st = x == 0 ? "ak" : "bk";
        if (kc[x]) o << "    " << v << " = *(const GM f4u*)(p" << nm[x] << " + " << 8 * gr << ");\n";
        else for (int t = 0; t < 4; ++t) o << "    " << v << "[" << t << "] = p" << nm[x] << "[" << 8 * gr + t << " * " << st << "];\n";
      }
    o << "    pA += " << 8 * groups << " * ak; pB += " << 8 * groups << " * bk;\n";
  };
  auto products = [&](const char* from, int groups) {
    for (int gr = 0; gr < groups; ++gr)
      for (int t = 0; t < 4; ++t) {
        const char* ac = t % 2 ? "acc2" : "acc";
        const std::string i = std::to_string(gr) + "[" + std::to_string(t) + "]";
        o << "    " << ac << " = __builtin_amdgcn_mfma_f32_32x32x2f32(" << from << "A" << i << ", " << from << "B" << i << ", " << ac << ", 0, 0, 0);\n";
      }
  };
  o << "  f4 ";
  for (const char* set : {"u", "v"}) for (int x = 0; x < 2; ++x) for (int gr = 0; gr < NK / 8; ++gr) o << (set[0] == 'u' && x == 0 && gr == 0 ? "" : ", ") << set << nm[x] << gr;
  o << ";\n  if (n >= " << NK << ") {\n";
  whole("u", NK / 8);
  // (two steps at a time, so that the next one's registers have names of their own)
  o << "    for (; k + " << 3 * NK << " <= n; k += " << 2 * NK << ") {\n";
  whole("v", NK / 8);
  products("u", NK / 8);
  whole("u", NK / 8);
  products("v", NK / 8);
  o << "    }\n    if (k + " << 2 * NK << " <= n) {\n";
  whole("v", NK / 8);
  products("u", NK / 8);
  products("v", NK / 8);
  o << "      k += " << 2 * NK << ";\n    } else {\n";
  products("u", NK / 8);
  o << "      k += " << NK << ";\n    }\n  }\n"
       // what is left: a whole group of eight, and positions of which those past the end are zero in both operands
       "  if (k + 8 <= n) {\n";
  whole("u", 1);
  products("u", 1);
  o << "    k += 8;\n  }\n  if (k < n) {\n    const int left = n - k - 4 * (int)lh;\n";
  for (int x = 0; x < 2; ++x)
    for (int t = 0; t < 4; ++t)
      o << "    { const float w = p" << nm[x] << "[(long long)(" << t << " < left ? " << t << " : left - 1) * " << (x == 0 ? "ak" : "bk") << "]; u" << nm[x] << "0[" << t << "] = " << t << " < left ? w : 0.0f; }\n";
  products("u", 1);
  o << "  }\n  acc += acc2;\n  GM float* const out = (GM float*)" << e.slot(e.L.out) << ";\n";
  if (KW == 1) {
    // a block inside the result stores without a look at every element
    o << "  GM float* const po = out + (m0 + 4 * lh) * N + n0 + l32;\n  const bool inside = m0 + 32 <= M && n0 + 32 <= N;\n";
    for (int guarded = 0; guarded < 2; ++guarded) {
      o << (guarded ? "  else {\n" : "  if (inside) {\n");
      const std::string body = captured(e, [&] {
        o << "#pragma unroll\n    for (int ql = 0; ql < 4; ++ql) {\n      const int q = 4 * qh + ql;\n"
             "      const long long row = m0 + 8 * qh + 4 * lh + ql, col = n0 + l32;\n" << (guarded ? "      if (row < M && col < N) {\n" : "      {\n") << "        const float cacc = acc[q];\n";
        emit_scalar_program(e, g.prog, g.results, epi_load, "cacc", "t", "        ");
        o << "        po[(8 * qh + ql) * N] = t" << g.results[0] << ";\n      }\n    }\n";
      });
      emit_unrolled(o, {{"qh", 4}}, body, "    ");
      o << "  }\n";
    }
  } else {
    o << "  __shared__ float sm[" << KW << "][1024];\n"
         "#pragma unroll\n  for (int q = 0; q < 16; ++q) sm[wave][q * 64 + lane] = acc[q];\n  __syncthreads();\n"
         "#pragma unroll\n  for (int i = 0; i < " << 16 / KW << "; ++i) {\n    const unsigned at = threadIdx.x + i * " << 64 * KW << ", q = at / 64, ln = at % 64;\n    float w[" << KW << "];\n"
         "#pragma unroll\n    for (int x = 0; x < " << KW << "; ++x) w[x] = sm[x][at];\n"
         "#pragma unroll\n    for (int d = 1; d < " << KW << "; d *= 2)\n#pragma unroll\n      for (int x = 0; x < " << KW << "; x += 2 * d) w[x] += w[x + d];\n"
         "    const long long row = m0 + 8 * (q / 4) + 4 * (ln / 32) + q % 4, col = n0 + ln % 32;\n"
         "    if (row < M && col < N) {\n      const float cacc = w[0];\n      if (NSPLIT > 1) ((GM float*)" << e.slot(e.L.ocoef) << ")[(split * M + row) * N + col] = cacc;\n      else {\n";
    emit_scalar_program(e, g.prog, g.results, epi_load, "cacc", "t", "        ");
    o << "        out[row * N + col] = t" << g.results[0] << ";\n      }\n    }\n  }\n";
  }
  o << "}\n";
}

// C = A.B for f32 on MFMA (v_mfma_f32_32x32x2_f32: f32 inputs, f32 accumulation), the one place
// on this path that is a dense contraction.  A workgroup of four waves owns a 128x128 tile of
// C; each wave a 64x64 quarter as 2x2 MFMA blocks (64 accumulator VGPRs).  K advances in steps
// of 16: the next A and B tiles are fetched from global memory into registers (dwordx4 along
// whichever dimension of the operand is contiguous, so transposed views cost nothing) while the
// current tiles are consumed from LDS, k-major so that the 32 lanes of an MFMA operand read 32
// consecutive words.  The pointwise consumers of the dot run on the accumulators (epilogue).
void gen_gemm(Em& e) {
  const GroupPlan& g = e.g;
  const AccessGroup& ag = g.groups[g.mat_group];
  const AccessGroup& bg = g.groups[g.vec_group];
  const int a_mode = ag.coef[1] == 1 ? 0 : (ag.coef[0] == 1 ? 1 : 2);  // 0: k contiguous, 1: m contiguous, 2: neither
  const int b_mode = bg.coef[1] == 1 ? 0 : (bg.coef[0] == 1 ? 1 : 2);  // 0: n contiguous, 1: k contiguous, 2: neither
  // Tile of C per workgroup: 128 x 128 (four waves, each a 64 x 64 quarter as 2 x 2 matrix-core
  // blocks), or 128 x 32 for products with at most 32 columns (each wave one 32 x 32 block of its
  // own 32 rows): a 128-wide tile would spend the matrix cores on columns that do not exist.
  const int BN = g.BX == 32 ? 32 : 128;
  const int IB = BN == 128 ? 2 : 1, JB = IB;   // 32 x 32 blocks per wave along m and n
  // padded LDS rows: k-major tiles of 128 (B: BN) floats.  An operand that is contiguous along k is
  // transposed on its way into LDS by scalar writes, four k rows apart within a wave: a row pitch of
  // 130 puts those rows eight banks apart (pitch 132: only two distinct bank offsets, every write a
  // two-way conflict); an operand copied row by row with 16-byte writes needs a multiple of four.
  // K advances in steps of KS = 16 (one barrier per step), or 32 on request (option "gemm_kstep";
  // measured slower: 127 against 134 TFLOP/s on 4096^3).
  const int KS = BN == 128 && g.UC == 2 ? 32 : 16;
  const int TK = KS / 4;        // threads along k of an operand that is contiguous along k (four floats each)
  const int NI = KS / 8;        // vector loads per thread and operand tile
  const int AP = a_mode == 0 ? (KS == 32 ? 129 : 130) : 132;
  const int BP = BN == 128 && b_mode == 1 ? (KS == 32 ? 129 : 130) : BN + 4;
  prelude(e);
  e.o << "typedef float f16v __attribute__((ext_vector_type(16)));\n";
  if (g.VR == 2 && g.UC == 2) split_helpers(e);
  kernel_head(e, "gr_gemm", gemm_threads(g));
  e.o << "  const long long M = " << e.S(e.L.extra) << ", N = " << e.S(e.L.extra + 1) << ", K = " << e.S(e.L.extra + 2) << ";\n";
  group_pointers(e, "  ");
  e.o << "  const GM float* const A = q" << g.mat_group << "; const GM float* const B = q" << g.vec_group << ";\n";
  e.o << "  const long long am = " << e.coef(g.mat_group, 0) << ", ak = " << e.coef(g.mat_group, 1) << ", bk = " << e.coef(g.vec_group, 0)
      << ", bn = " << e.coef(g.vec_group, 1) << ";\n  (void)am; (void)ak; (void)bk; (void)bn;\n";
  const EpiLoad epi_load = [&](const Instr& in, int) {
    const AccessGroup& eg = g.groups[in.group];
    std::ostringstream s2;
    s2 << e.qp << in.group << "[0";
    if (!eg.structural_zero[0]) s2 << " + (row + " << in.delta[0] << ") * " << e.coef(in.group, 0);
    if (!eg.structural_zero[1]) s2 << " + (col + " << in.delta[1] << ") * " << e.coef(in.group, 1);
    s2 << "]";
    return s2.str();
  };
  auto emit_combine = [&]() { gemm_combine(e, epi_load); };
  if (g.VR == 4) {   // blocks of 32 x 32 from registers
    gemm_block_body(e, epi_load);
    emit_combine();
    return;
  }
  if (g.VR == 3) {   // small tiles, clamped loads
    gemm_tile_body(e, epi_load);
    emit_combine();
    return;
  }
  if (g.VR == 2) {   // tiles loaded straight into LDS
    gemm_big_body(e, epi_load);
    emit_combine();
    return;
  }
  e.o << "  __shared__ float As[2][" << KS << "][" << AP << "];\n  __shared__ float Bs[2][" << KS << "][" << BP << "];\n";
  e.o << "  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;\n";
  if (BN == 128) e.o << "  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64, l32 = lane & 31, lh = lane >> 5;\n";
  else e.o << "  const int wm = wave * 32, wn = 0, l32 = lane & 31, lh = lane >> 5;\n";
  // split-K for products with few output tiles: workgroup (tile, split) accumulates k in
  // [kbeg, KE) and leaves its partial tile in a workspace; gr_gemm_combine adds the partial tiles
  // in a fixed order and applies the epilogue (the two-kernel reduction of Section 3.2)
  e.o << "  const long long NSPLIT = " << e.S(e.L.extra + 3) << ", KCH = " << e.S(e.L.ocoef + 1) << ";\n";
  e.o << "  const long long tiles_n = (N + " << BN - 1 << ") / " << BN << ", tiles = tiles_n * ((M + 127) / 128);\n";
  e.o << "  const long long tile = blockIdx.x % tiles, split = blockIdx.x / tiles;\n";
  e.o << "  const long long bm0 = (tile / tiles_n) * 128, bn0 = (tile % tiles_n) * " << BN << ";\n";
  e.o << "  const long long kbeg = split * KCH, KE = (kbeg + KCH < K) ? kbeg + KCH : K;\n";
  e.o << "  f16v acc[" << IB << "][" << JB << "];\n  for (int i = 0; i < " << IB << "; ++i) for (int j = 0; j < " << JB << "; ++j) for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.0f;\n";
  e.o << "  float ra[" << 4 * NI << "], rb[" << 4 * NI << "];\n  (void)rb;\n";
  // --- global -> registers, per operand a guarded version (edge tiles, K tail) and an unguarded
  // one for tiles that lie inside the operand: straight-line loads that the compiler keeps in
  // flight under the matrix instructions of the previous step
  for (int guarded = 1; guarded >= 0; --guarded) {
    e.o << "  auto fetchA" << (guarded ? "_g" : "_u") << " = [&](long long k0) {\n";
    if (a_mode == 0) {
      e.o << "    for (int i = 0; i < " << NI << "; ++i) {\n      const long long row = bm0 + tid / " << TK << " + " << 256 / TK << " * i, kk = k0 + (tid % " << TK << ") * 4;\n";
      if (guarded) e.o << "      if (row < M && kk + 4 <= KE) { const f4u w = *(const GM f4u*)(A + row * am + kk); ra[4*i] = w[0]; ra[4*i+1] = w[1]; ra[4*i+2] = w[2]; ra[4*i+3] = w[3]; }\n"
                          "      else { for (int j = 0; j < 4; ++j) ra[4*i+j] = (row < M && kk + j < KE) ? A[row * am + kk + j] : 0.0f; }\n    }\n";
      else e.o << "      const f4u w = *(const GM f4u*)(A + row * am + kk); ra[4*i] = w[0]; ra[4*i+1] = w[1]; ra[4*i+2] = w[2]; ra[4*i+3] = w[3];\n    }\n";
    } else if (a_mode == 1) {
      e.o << "    for (int i = 0; i < " << NI << "; ++i) {\n      const long long kk = k0 + tid / 32 + 8 * i, row = bm0 + (tid % 32) * 4;\n";
      if (guarded) e.o << "      if (kk < KE && row + 4 <= M) { const f4u w = *(const GM f4u*)(A + kk * ak + row); ra[4*i] = w[0]; ra[4*i+1] = w[1]; ra[4*i+2] = w[2]; ra[4*i+3] = w[3]; }\n"
                          "      else { for (int j = 0; j < 4; ++j) ra[4*i+j] = (kk < KE && row + j < M) ? A[kk * ak + row + j] : 0.0f; }\n    }\n";
      else e.o << "      const f4u w = *(const GM f4u*)(A + kk * ak + row); ra[4*i] = w[0]; ra[4*i+1] = w[1]; ra[4*i+2] = w[2]; ra[4*i+3] = w[3];\n    }\n";
    } else {
      e.o << "    for (int i = 0; i < " << 4 * NI << "; ++i) { const int el = tid + 256 * i; const long long row = bm0 + el % 128, kk = k0 + el / 128;\n";
      if (guarded) e.o << "      ra[i] = (row < M && kk < KE) ? A[row * am + kk * ak] : 0.0f; }\n";
      else e.o << "      ra[i] = A[row * am + kk * ak]; }\n";
    }
    e.o << "  };\n";
    e.o << "  auto fetchB" << (guarded ? "_g" : "_u") << " = [&](long long k0) {\n";
    if (BN == 32) {
      // 16 x 32 tile: two elements per thread, always guarded (the operand is small)
      e.o << "    for (int i = 0; i < 2; ++i) { const int el = tid + 256 * i; const long long col = bn0 + el % 32, kk = k0 + el / 32;\n"
             "      rb[i] = (col < N && kk < KE) ? B[kk * bk + col * bn] : 0.0f; }\n";
    } else if (b_mode == 0) {
      e.o << "    for (int i = 0; i < " << NI << "; ++i) {\n      const long long kk = k0 + tid / 32 + 8 * i, col = bn0 + (tid % 32) * 4;\n";
      if (guarded) e.o << "      if (kk < KE && col + 4 <= N) { const f4u w = *(const GM f4u*)(B + kk * bk + col); rb[4*i] = w[0]; rb[4*i+1] = w[1]; rb[4*i+2] = w[2]; rb[4*i+3] = w[3]; }\n"
                          "      else { for (int j = 0; j < 4; ++j) rb[4*i+j] = (kk < KE && col + j < N) ? B[kk * bk + col + j] : 0.0f; }\n    }\n";
      else e.o << "      const f4u w = *(const GM f4u*)(B + kk * bk + col); rb[4*i] = w[0]; rb[4*i+1] = w[1]; rb[4*i+2] = w[2]; rb[4*i+3] = w[3];\n    }\n";
    } else if (b_mode == 1) {
      e.o << "    for (int i = 0; i < " << NI << "; ++i) {\n      const long long col = bn0 + tid / " << TK << " + " << 256 / TK << " * i, kk = k0 + (tid % " << TK << ") * 4;\n";
      if (guarded) e.o << "      if (col < N && kk + 4 <= KE) { const f4u w = *(const GM f4u*)(B + col * bn + kk); rb[4*i] = w[0]; rb[4*i+1] = w[1]; rb[4*i+2] = w[2]; rb[4*i+3] = w[3]; }\n"
                          "      else { for (int j = 0; j < 4; ++j) rb[4*i+j] = (col < N && kk + j < KE) ? B[col * bn + kk + j] : 0.0f; }\n    }\n";
      else e.o << "      const f4u w = *(const GM f4u*)(B + col * bn + kk); rb[4*i] = w[0]; rb[4*i+1] = w[1]; rb[4*i+2] = w[2]; rb[4*i+3] = w[3];\n    }\n";
    } else {
      e.o << "    for (int i = 0; i < " << 4 * NI << "; ++i) { const int el = tid + 256 * i; const long long col = bn0 + el % 128, kk = k0 + el / 128;\n";
      if (guarded) e.o << "      rb[i] = (col < N && kk < KE) ? B[kk * bk + col * bn] : 0.0f; }\n";
      else e.o << "      rb[i] = B[kk * bk + col * bn]; }\n";
    }
    e.o << "  };\n";
  }
  // --- registers -> LDS (k-major tiles), in pieces: a piece is what one of a thread's vector loads brought
  // (four floats of A or of B).  The main loop puts one piece behind each of the last matrix
  // instructions of a step, so that the LDS writes are issued while the matrix cores work; all of
  // them in a row after the last matrix instruction cost a tenth of the kernel's time (measured).
  std::vector<std::string> pieces;
  for (int i = 0; i < NI; ++i) {
    const std::string I = std::to_string(i);
    if (a_mode == 0) pieces.push_back("for (int j = 0; j < 4; ++j) As[buf][(tid % " + std::to_string(TK) + ") * 4 + j][tid / " + std::to_string(TK) + " + " + std::to_string(256 / TK) + " * " + I + "] = ra[4*" + I + "+j];");
    else if (a_mode == 1) pieces.push_back("for (int j = 0; j < 4; ++j) As[buf][tid / 32 + 8 * " + I + "][(tid % 32) * 4 + j] = ra[4*" + I + "+j];");
    else pieces.push_back("for (int i = " + std::to_string(4 * i) + "; i < " + std::to_string(4 * i + 4) + "; ++i) { const int el = tid + 256 * i; As[buf][el / 128][el % 128] = ra[i]; }");
  }
  if (BN == 32) pieces.push_back("for (int i = 0; i < 2; ++i) { const int el = tid + 256 * i; Bs[buf][el / 32][el % 32] = rb[i]; }");
  else for (int i = 0; i < NI; ++i) {
    const std::string I = std::to_string(i);
    if (b_mode == 0) pieces.push_back("for (int j = 0; j < 4; ++j) Bs[buf][tid / 32 + 8 * " + I + "][(tid % 32) * 4 + j] = rb[4*" + I + "+j];");
    else if (b_mode == 1) pieces.push_back("for (int j = 0; j < 4; ++j) Bs[buf][(tid % " + std::to_string(TK) + ") * 4 + j][tid / " + std::to_string(TK) + " + " + std::to_string(256 / TK) + " * " + I + "] = rb[4*" + I + "+j];");
    else pieces.push_back("for (int i = " + std::to_string(4 * i) + "; i < " + std::to_string(4 * i + 4) + "; ++i) { const int el = tid + 256 * i; Bs[buf][el / 128][el % 128] = rb[i]; }");
  }
  e.o << "  auto stash = [&](int buf) {\n";
  for (const std::string& pc : pieces) e.o << "    " << pc << "\n";
  e.o << "  };\n";
  if (BN == 128) {
    // The operands of matrix-instruction group ks + 1 are read from LDS before the four matrix
    // instructions of group ks are issued: the reads complete under 256 cycles of matrix work
    // (measured on 4096^3: 127 -> 133.7 TFLOP/s), and one piece of the next tile goes to LDS behind
    // each of the last matrix instructions of the step.  Scheduling barriers keep the order written
    // here: the compiler's scheduler would sink the reads below the matrix instructions and gather
    // the LDS writes at the end.  (A pure matrix-instruction loop reaches 155.6 TFLOP/s on this
    // device.  Measured and not adopted: steps of 32 values of k, 127 TFLOP/s; two barriers per
    // step with the LDS writes in the first half and the first operands of the next step read
    // before the second barrier, 132.6; a second or third resident workgroup per compute unit,
    // workgroups started half a step apart: no change.)
    const int G = KS / 2;                                   // groups of four matrix instructions per step
    const int first = G * 4 - 1 - (int)pieces.size();       // matrix instruction (0-based, of 4G) after which the first piece goes; none after the last
    e.o << "  auto step = [&](int cur, bool more) {\n"
           "    const int buf = cur ^ 1;\n"
           "    float a0 = As[cur][lh][wm + l32], a1 = As[cur][lh][wm + 32 + l32];\n"
           "    float b0 = Bs[cur][lh][wn + l32], b1 = Bs[cur][lh][wn + 32 + l32];\n";
    for (int ks = 0; ks < G; ++ks) {
      e.o << "    {\n      float na0 = 0.0f, na1 = 0.0f, nb0 = 0.0f, nb1 = 0.0f;\n";
      if (ks < G - 1)
        e.o << "      na0 = As[cur][" << 2 * ks + 2 << " + lh][wm + l32]; na1 = As[cur][" << 2 * ks + 2 << " + lh][wm + 32 + l32];\n"
               "      nb0 = Bs[cur][" << 2 * ks + 2 << " + lh][wn + l32]; nb1 = Bs[cur][" << 2 * ks + 2 << " + lh][wn + 32 + l32];\n";
      e.o << "      __builtin_amdgcn_sched_barrier(0);\n";
      const char* mm[4] = {"acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b0, acc[0][0], 0, 0, 0);", "acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b1, acc[0][1], 0, 0, 0);",
                           "acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b0, acc[1][0], 0, 0, 0);", "acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b1, acc[1][1], 0, 0, 0);"};
      for (int m = 0; m < 4; ++m) {
        e.o << "      " << mm[m] << "\n";
        const int pi = ks * 4 + m - first;
        if (pi >= 0 && pi < (int)pieces.size())
          e.o << "      __builtin_amdgcn_sched_barrier(0);\n      if (more) { " << pieces[pi] << " }\n      __builtin_amdgcn_sched_barrier(0);\n";
      }
      e.o << "      a0 = na0; a1 = na1; b0 = nb0; b1 = nb1;\n    }\n";
    }
    e.o << "  };\n";
  } else
    e.o << "  auto step = [&](int cur, bool more) {\n#pragma unroll\n    for (int ks = 0; ks < 8; ++ks) {\n"
           "      const float a0 = As[cur][2 * ks + lh][wm + l32];\n"
           "      const float b0 = Bs[cur][2 * ks + lh][l32];\n"
           "      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b0, acc[0][0], 0, 0, 0);\n    }\n"
           "    if (more) stash(cur ^ 1);\n  };\n";
  e.o << "  const long long nkt = KE > kbeg ? (KE - kbeg + " << KS - 1 << ") / " << KS << " : 0;\n  int cur = 0;\n";
  // workgroup-uniform choice between four loops: each operand unguarded where its tile is interior
  e.o << "  const bool kfull = (KE - kbeg) % " << KS << " == 0, a_in = kfull && bm0 + 128 <= M, b_in = kfull && bn0 + " << BN << " <= N;\n";
  auto loop = [&](const char* fa, const char* fb, const char* ind) {
    e.o << ind << "if (nkt > 0) { " << fa << "(kbeg); " << fb << "(kbeg); stash(0); }\n" << ind << "__syncthreads();\n"
        << ind << "for (long long kt = 0; kt < nkt; ++kt) {\n"
        << ind << "  if (kt + 1 < nkt) { " << fa << "(kbeg + (kt + 1) * " << KS << "); " << fb << "(kbeg + (kt + 1) * " << KS << "); }\n"
        << ind << "  step(cur, kt + 1 < nkt);\n"
        << ind << "  __syncthreads();\n" << ind << "  cur ^= 1;\n" << ind << "}\n";
  };
  e.o << "  if (a_in && b_in) {\n";
  loop("fetchA_u", "fetchB_u", "    ");
  e.o << "  } else if (a_in) {\n";
  loop("fetchA_u", "fetchB_g", "    ");
  e.o << "  } else if (b_in) {\n";
  loop("fetchA_g", "fetchB_u", "    ");
  e.o << "  } else {\n";
  loop("fetchA_g", "fetchB_g", "    ");
  e.o << "  }\n";
  // --- epilogue on the accumulators: element q of a 32x32 block sits at row 8*(q/4) + 4*(lane/32) + q%4, column lane%32
  e.o << "  GM float* const out = (GM float*)" << e.slot(e.L.out) << ";\n";
  e.o << "  if (NSPLIT > 1) {\n    GM float* const ws = (GM float*)" << e.slot(e.L.ocoef) << " + split * M * N;\n"
         "#pragma unroll\n    for (int i = 0; i < " << IB << "; ++i)\n#pragma unroll\n    for (int j = 0; j < " << JB << "; ++j)\n#pragma unroll\n      for (int q = 0; q < 16; ++q) {\n"
         "        const long long row = bm0 + wm + 32 * i + 8 * (q / 4) + 4 * lh + (q % 4), col = bn0 + wn + 32 * j + l32;\n"
         "        if (row < M && col < N) ws[row * N + col] = acc[i][j][q];\n      }\n    return;\n  }\n";
  // (an index of acc that is not a constant would move the accumulators to scratch memory: the loops over blocks
  // and over groups of four elements are unrolled in the text, the four elements of a group by the compiler)
  const std::string body = captured(e, [&] {
    e.o << "#pragma unroll\n      for (int ql = 0; ql < 4; ++ql) {\n"
           "      const int q = 4 * qh + ql;\n"
           "      const long long row = bm0 + wm + 32 * i + 8 * qh + 4 * lh + ql, col = bn0 + wn + 32 * j + l32;\n"
           "      if (row < M && col < N) {\n        const float cacc = acc[i][j][q];\n";
    emit_scalar_program(e, g.prog, g.results, epi_load, "cacc", "t", "        ");
    e.o << "        out[row * N + col] = t" << g.results[0] << ";\n      }\n      }\n";
  });
  emit_unrolled(e.o, {{"i", IB}, {"j", JB}, {"qh", 4}}, body, "    ");
  e.o << "}\n";
  emit_combine();
}

// The second kernel of a matrix product whose K range is split over workgroups.
void gemm_combine(Em& e, const EpiLoad& epi_load) {
  const GroupPlan& g = e.g;
  // second stage of a split product: partial tiles added in split order, then the epilogue
  kernel_head(e, "gr_gemm_combine");
  e.o << "  const long long M = " << e.S(e.L.extra) << ", N = " << e.S(e.L.extra + 1) << ", NSPLIT = " << e.S(e.L.extra + 3) << ";\n";
  e.o << "  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;\n  if (idx >= M * N) return;\n";
  e.o << "  const long long row = idx / N, col = idx % N;\n";
  e.o << "  const GM float* const ws = (const GM float*)" << e.slot(e.L.ocoef) << ";\n";
  e.o << "  GM float* const out = (GM float*)" << e.slot(e.L.out) << ";\n";
  group_pointers(e, "  ", {g.mat_group, g.vec_group});
  e.o << "  float cacc = ws[idx];\n  long long s = 1;\n"
         "  for (; s + 4 <= NSPLIT; s += 4) {\n"
         "    const float v0 = ws[s * M * N + idx], v1 = ws[(s + 1) * M * N + idx], v2 = ws[(s + 2) * M * N + idx], v3 = ws[(s + 3) * M * N + idx];\n"
         "    cacc = (((cacc + v0) + v1) + v2) + v3;\n  }\n"
         "  for (; s < NSPLIT; ++s) cacc += ws[s * M * N + idx];\n";
  emit_scalar_program(e, g.prog, g.results, epi_load, "cacc", "t", "  ");
  e.o << "  out[idx] = t" << g.results[0] << ";\n}\n";
}

}  // namespace

std::string generate_source(const GroupPlan& g) {
  Em e(g);
  switch (g.kind) {
    case GroupKind::MAP: if (g.in_place) gen_map_in_place(e); else gen_map(e); break;
    case GroupKind::ROWRED: gen_rowred(e); break;
    case GroupKind::REDUCE:
      if (g.pair) {
        Em e2(*g.pair);
        e2.slot_base = e.L.total;
        e.total_slots = e.L.total + e2.L.total;
        gen_reduce(e, e2.slot(e2.L.out));
      } else gen_reduce(e);
      break;
    case GroupKind::SCAN: gen_scan(e); break;
    case GroupKind::GEMM: gen_gemm(e); break;
    case GroupKind::GEMV:
      if (g.gemv_mode == 2) {
        Em e2(*g.pair);
        e2.slot_base = e.L.total;
        e.total_slots = e2.total_slots = e.L.total + e2.L.total;
        gen_gemv_pair(e, e2);
      } else if (g.gemv_mode == 1) gen_gemv_colacc(e);
      else gen_gemv_rowdot(e);
      break;
  }
  return e.o.str();
}

}  // namespace gr
