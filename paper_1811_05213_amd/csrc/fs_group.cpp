// fs_group.cpp - fused-group analysis, schedule and LDS planning, and group formation.
#include <algorithm>
#include <functional>
#include <set>
#include <cstdlib>

#include "fs_internal.h"

namespace fs {

namespace {

// Do column tiles, which are walked tile by tile, share cache lines with their neighbours at most rows?  8 neighbours then run on one XCD.  Batch
// normalisation fp32 [16384,1001] 41.0 -> 38.0 us, [8192,2001] 40.6 -> 36.5, [1000,4001] 12.6 -> 11.7, [30000,517] 42.2 -> 41.2; column sums beside row norms
// [1500,2001] 12.5 -> 10.8, [3440,1000] 11.3 -> 10.4.  Not for rows of whole lines ([16384,1024] 26.8 against 29.0), nor for a few tiles or
// workgroups, which part the rows instead ([56203,143] 31.7 against 33.4).
bool tiles_share_lines(const GroupPlan& gp) {
  bool shared = false;
  for (const auto* list : {&gp.ext_in, &gp.ext_out})
    for (const ExtTensor& e : *list) shared |= e.kind == KIND_FULL && (int64_t)gp.C * dtype_size(e.dtype) % 128 != 0;
  return shared && gp.s.CT >= 5 && gp.s.grid >= 64;
}

// How long workgroups wait for each other: several times what those of the largest kernels need from their start to the last load.  Joined
// kernels 50 us, before they do each other's work.  Column folds 100 us, before they leave the rest to the last one: beside a streaming
// kernel of another stream LayerNorm backward fp32 [8192,4096] takes 209 us with that, 225 with 50 us, 232 with 20 (201 with the tree), moments
// [16384,2048] 178, 216, 261 (183); [5000,3000] beside a long softmax 102, 113, 216 (102).
int wait_ticks(int ticks) {
  const char* e = getenv("FS_JOIN_WAIT_TICKS");
  return e ? atoi(e) : ticks;
}

int pow2_floor(int x) {
  int p = 1;
  while (p * 2 <= x) p *= 2;
  return p;
}
int pow2_ceil(int x) {
  int p = 1;
  while (p < x && p < (1 << 30)) p <<= 1;
  return p;
}

struct Resolved {
  bool literal = false;  // FS_CONST: no tensor behind it
  int node = -1;         // the tensor actually read (bcasts looked through)
  Kind kind = KIND_NONE; // its kind in the group's work space
};

struct Analyser {
  const Graph& g;
  GroupPlan& gp;
  std::vector<char> in_set;
  int R = 1, C = 1;

  Analyser(const Graph& g_, GroupPlan& gp_) : g(g_), gp(gp_), in_set(g_.n(), 0) {}

  Kind classify(int rows, int cols) const {
    if (rows == R && cols == C) return KIND_FULL;
    if (rows == R && cols == 1) return KIND_COLV;
    if (rows == 1 && cols == C) return KIND_ROWV;
    return KIND_NONE;
  }
  // t: the tensor lives in the transposed orientation of the work space (its [r,c] is the work
  // space's [c,r]).  A [C,1] tensor of that orientation is one value per work-space column and has
  // the memory layout of a [1,C] tensor, so vectors need no data movement at all.
  Kind classify(const fs_node& n, bool t) const { return t ? classify(n.cols, n.rows) : classify(n.rows, n.cols); }

  int source_of(int o) const {
    const fs_node& n = g.nodes[o];
    return (n.opcode == FS_BCAST_ROWVEC || n.opcode == FS_BCAST_COLVEC) ? n.in[0] : o;
  }

  // What a consumer working in orientation t and expecting kind `want` sees when it reads operand `o`.
  bool resolve(int o, Kind want, bool t, Resolved* r) const {
    const fs_node& n = g.nodes[o];
    if (classify(n, t) != want) return false;
    if (n.opcode == FS_CONST) {
      r->literal = true;
      return true;
    }
    if (n.opcode == FS_BCAST_ROWVEC || n.opcode == FS_BCAST_COLVEC) {
      const int x = n.in[0];
      const fs_node& xn = g.nodes[x];
      if (xn.opcode == FS_CONST) {
        r->literal = true;
        return true;
      }
      const Kind kx = classify(xn, t);
      if (kx == KIND_NONE) return false;
      // a broadcast either widens a vector to the full work space or is the identity
      const Kind vec = ((n.opcode == FS_BCAST_ROWVEC) != t) ? KIND_ROWV : KIND_COLV;
      if (!(kx == want || (want == KIND_FULL && kx == vec))) return false;
      r->node = x;
      r->kind = kx;
      return true;
    }
    r->node = o;
    r->kind = want;
    return true;
  }
};

// [R,C] tensors far larger than the caches
constexpr uint64_t kStreamBytes = 32ull << 20;

void add_ext_in(GroupPlan& gp, int node, Kind k, int dtype) {
  for (const ExtTensor& e : gp.ext_in)
    if (e.node == node) return;
  ExtTensor e;
  e.node = node;
  e.kind = k;
  e.dtype = dtype;
  gp.ext_in.push_back(e);
}

}  // namespace

// -------------------------------------------------------------------------------------------
// Schedule and LDS plan of one group.
//
// Every group runs a Row schedule with split_dim = 0 (Section 4.1): the work space [R,C] is
// cut along rows into `grid` blocks.  What is tuned is how many lanes cooperate on a row (L,
// the role of reduce_warps in Section 4.4), the workgroup size and the block count.  Row
// reductions want a row inside one wavefront (no LDS, no barrier); very long rows are spread
// over several wavefronts and folded through LDS; small problems trade elements per lane
// for more wavefronts so that the 256 CUs all get work.
// -------------------------------------------------------------------------------------------
namespace {
constexpr int kNarrowRegs = 96;  // registers a lane of a narrow column tile may hold in rows, accumulators and [1,C] operands

// The decisions of one group's schedule, taken in a fixed order; every step reads what the steps before it decided.
struct Scheduler {
  const Graph& g;
  const PlanOptions& opt;
  GroupPlan* gp;
  Schedule& s;
  const int R, C;
  // the machine: compute units and resident lanes as the device reports them (256 and 524288 on MI355X)
  int CUS = 0;
  int64_t RES = 0;
  // what the group is made of
  int max_es = 0, V = 4, NV = 0;
  bool has_concat = false, rowred = false, colred = false, has_transposed = false, tileable = false;
  // the form its rows take
  int ecap = 8, l_min = 1, l_max = 1, l_hint = 1;  // (l_hint: the fewest lanes per row a hint may ask for)
  bool few_long_rows = false, split_rows = false, resident = false, chunked = false, col_tiled = false, narrow_tiles = false, tiled_transpose = false;
  // lanes, vectors, workgroup
  int narrow_lanes = 0, narrow_trip_regs = 0, narrow_regs = 0;  // narrow column tiles: lanes, registers a trip's rows take, and accumulators and [1,C] operands
  int L = 64, tt_rows = 64, NVL = 1, CT = 1, NVLC = 0, RESV = 0, WG = 256;
  int lead = 0;  // rows are held in pieces of whole lines of this many elements (lead_rows)
  bool in_pairs = false;  // rows are read two elements at a time (pick_vector_width)
  bool staged_loop = false;
  int row_inputs = 0;        // [R,C] tensors from memory
  bool whole_lanes = true;   // ... of which a lane takes 16 bytes at a time

  Scheduler(const Graph& g_, const PlanOptions& opt_, GroupPlan* gp_) : g(g_), opt(opt_), gp(gp_), s(gp_->s), R(gp_->rows()), C(gp_->cols()) {}

  // lanes per row are a power of two: when half as many lanes would hold the row with at most
  // 1.5 x a cap below 32, take them (5120 bf16 columns under a cap of 16: 256 lanes x 24 elements,
  // not 512 x 16 with 37 % of the lanes idle)
  int lanes_for(int e) const {
    const int l = pow2_ceil((NV + e / V - 1) / (e / V));
    if (rowred && l >= 2 && e < 32 && ((NV + l / 2 - 1) / (l / 2)) * V * 2 <= e * 3) return l / 2;
    return l;
  }

  // whether a hint asks for several row tiles a trip: rows in pieces of whole lines and rows asked for ahead come one tile at a time
  bool several_tiles() const { return opt.has_hint && opt.hint.tiles_per_trip >= 2 && opt.hint.tiles_per_trip <= 4; }

  // lanes per row that a hint asks for, 0 when it asks for none or for what the group cannot have
  int hinted_lanes() const {
    const int h = opt.has_hint ? opt.hint.lanes_per_row : 0;
    return h > 0 && (h & (h - 1)) == 0 && h >= l_hint && h <= 1024 ? h : 0;
  }

  // 2-D transpose tiles keep the shape that measured best whatever a hint asks, but for tensors of up to 256 columns, whose tiles
  // hardly differ from whole rows: there lanes and workgroup are worth tuning
  bool tile_hints() const { return C <= 256; }

  // element size, vector width, which reductions the group holds
  fs_status measure_group() {
    // the machine: compute units and resident lanes as the device reports them (256 and 524288 on MI355X)
    CUS = device_limits().cus;
    RES = device_limits().resident_lanes;
    max_es = 0;
    for (const ExtTensor& e : gp->ext_in)
      if (e.kind == KIND_FULL || e.kind == KIND_PART) max_es = std::max(max_es, dtype_size(e.dtype));
    for (const ExtTensor& e : gp->ext_out)
      if (e.kind == KIND_FULL) max_es = std::max(max_es, dtype_size(e.dtype));
    if (max_es == 0) max_es = 4;
    V = 16 / max_es;
    has_concat = false;
    for (int m : gp->members) has_concat |= g.nodes[m].opcode == FS_CONCAT;
    // A width that V does not divide keeps 16-byte accesses: the last vector of a row overlaps the one before it (fs_vec_col).
    // Rows of at most 32 bytes belong to one lane each and are read element by element or in the vectors that fit.  A vector
    // access must not straddle the seam of a concat, so there V divides the widths, as it does where whole rows of less than 16
    // elements leave transposed.
    bool narrow_transposed = false;
    for (const ExtTensor& e : gp->ext_out) narrow_transposed |= e.transposed && C < 16;
    // So it does where row sums are one link of a chain of launch-bound kernels: the vector width decides the order of a sum, and
    // what follows may cancel and amplify the last bits (outputs of the 200-node DAG at odd sizes: two orders of the same sums
    // differ by up to 3e-5 of an output's rms, both as far from float64).  Such kernels are chains of latencies and gain little
    // from wider accesses: DAG of [512,100] 26.6 -> 26.6 us, [333,256] 29.9 -> 27.7, [2047,384] (19 MB a kernel) 81.4 -> 78.4 us.
    // A kernel that holds its whole plan keeps them ([60000,65] fp32 softmax 30.1 -> 8.4 us, [256,1001] 3.5 -> 3.0 us), and
    // so does one that streams 32 MB or more.
    const bool keeps_order = !gp->row_reduces.empty() && gp->exchanges && gp->min_hbm_bytes < kStreamBytes;
    while (has_concat || narrow_transposed || keeps_order || (int64_t)C * max_es <= 32 ? C % V != 0 : V > C) V /= 2;
    for (int m : gp->members)
      if (g.nodes[m].opcode == FS_CONCAT && g.nodes[m].attr_i == FS_CONCAT_COLS)
        while (g.nodes[g.nodes[m].in[0]].cols % V) V /= 2;
    NV = C / V + (C % V != 0);
    rowred = !gp->row_reduces.empty();
    colred = !gp->col_reduces.empty();
    return FS_OK;
  }

  // Vectors that a width does not fill cost arithmetic as well as bytes: a lane computes on what its empty slots repeat.  Rows
  // with transcendental functions take pairs of elements instead where that leaves an eighth of the slots or more out.
  // bf16 (a 4-byte access each): masked softmax [4000,577] (1024 slots a row, 640 in pairs; element by element 5.2 us) 6.4 -> 4.7 us,
  // [6387,289] 5.7 -> 4.5, [16384,577] 11.4 -> 9.9, softmax [80000,577] 49.7 -> 44.6, [1500,4099] 5.8 -> 4.9.
  // fp32 below 40 MB: masked softmax [1817,577] 5.2 -> 4.7, [476,2201] 5.2 -> 4.7, softmax [694,6225] 8.2 -> 7.2, [682,2305] 4.6 -> 4.3
  // (at 60 MB [2382,3301] 10.7 -> 11.6, [1263,6225] 11.0 -> 11.7; beyond 8192 columns [604,13001] 11.8 -> 12.4).
  // Not without such functions (bf16 L2 normalisation [43000,289] 10.2 -> 10.6 us, row sums 8.9 -> 13.1), not with [1,C] operands, whose
  // slices take more accesses too (LayerNorm+GeLU [4700,577] 5.2 -> 5.7), not for short rows (bf16 [200000,65] 13.8 -> 15.7, fp32
  // [8004,131] 4.3 -> 4.6) or beyond 32 elements per lane (bf16 [1323,33001] 76.2 -> 81.7).
  fs_status pick_vector_width() {
    bool heavy = false, rowv = false;
    for (int m : gp->members) {
      const int op = g.nodes[m].opcode;
      heavy |= gp->kind.at(m) == KIND_FULL && (op == FS_EXP || op == FS_LOG || op == FS_TANH || op == FS_SIGMOID || op == FS_GELU_TANH);
    }
    for (const ExtTensor& e : gp->ext_in) rowv |= e.kind == KIND_ROWV;
    if (!heavy || rowv || V != 16 / max_es || V < 4 || C % V == 0 || !rowred || colred || has_transposed || chunked || CT > 1) return FS_OK;
    if (max_es == 2 ? C <= 128 || C > 32768 : C <= 256 || C > 8192 || gp->min_hbm_bytes >= (40u << 20)) return FS_OK;
    const int slots = NVL * L * V;
    for (int v : {2, V}) {
      V = v;
      NV = C / V + (C % V != 0);
      fs_status st;
      if ((st = pick_row_form()) != FS_OK || (st = pick_lanes()) != FS_OK || (st = pick_vectors()) != FS_OK) return st;
      in_pairs = V == 2 && !chunked && CT == 1 && NVL * L * V * 8 <= slots * 7;
      if (in_pairs) break;
    }
    return FS_OK;
  }

  // how a row is held: registers (16, 32, 64 elements per lane), a resident part plus chunks, chunks only, split over workgroups, column tiles, 2-D transpose tiles
  fs_status pick_row_form() {
    // Elements of one [R,C] value a lane may hold.  With row reductions the row stays in registers
    // across the stages together with everything else that is live: the other [R,C] inputs and the
    // lane's slices of the [1,C] operands (E registers each).  128 registers per lane keep four
    // wavefronts per SIMD in flight; 16 elements per lane is the most that pays even when more would
    // fit (measured over 26 row-reduction cases: 16 beats 32 by 3-10 %: more wavefronts per row, more
    // rows in flight); rows too long for that take 32 and 64 below.
    int n_live = 1;
    for (const ExtTensor& e : gp->ext_in) n_live += e.kind == KIND_FULL || e.kind == KIND_ROWV;
    n_live += (int)gp->col_reduces.size();  // a column accumulator per element
    ecap = rowred ? std::max(8, std::min(16, pow2_floor(128 / n_live))) : 8;
    if (colred && !rowred) ecap = 32 / max_es;  // 32 bytes per lane per tile (bf16 sums: 30.2 -> 25.4 us on [65536,1024])
    ecap = std::max(ecap, V);
    l_min = lanes_for(ecap);
    l_max = std::min(1024, pow2_ceil(NV));
    // Groups without reductions do not need a whole row in one workgroup: very long rows are cut
    // into column tiles, each handled like a row of its own.
    tileable = !rowred && !colred;
    has_transposed = false;
    for (const ExtTensor& e : gp->ext_out) has_transposed |= e.transposed;
    // A few very long rows occupy as many CUs as there are rows ([4, 4M] row sums: 263 us on 4 CUs).
    // When every row reduction of the group is in its first stage and everything else that leaves the
    // group is either a per-row value or computed before any reduction result, each row is split
    // over many workgroups; other such groups are better cut into kernels of that form and
    // reduction-free ones (worth_fusing).
    few_long_rows = rowred && !colred && !has_transposed && R <= 128 && (int64_t)C * max_es >= (1 << 18) && (int64_t)R * C * max_es >= (1 << 20);
    split_rows = few_long_rows;
    if (split_rows) {
      for (const ExtTensor& e : gp->ext_out) split_rows &= e.kind == KIND_COLV || gp->level.at(e.node) == 0;
      for (int m : gp->row_reduces) split_rows &= gp->level.at(m) == 0;
    }
    // Rows too long for that: first more elements per lane (32, then 64: one workgroup per CU, but the
    // row is still read once instead of once per stage); beyond that the first 48 (or 32) elements
    // per lane stay resident and the rest of the row is walked in chunks; last, chunks only.  Plan
    // creation steps `wide_level` down while the compiled kernel spills.
    // Rows whose [1,C] operands weigh at least as much per column as the rows themselves (LayerNorm with gamma, beta and a
    // bias over bf16 rows: 12 bytes against 4) keep nothing resident: their last stage needs the registers for the operands,
    // and the whole row fits LDS in its own dtype more often than not.  Measured, LayerNorm+GeLU bf16: [4096,65536] 323 us
    // with a resident part, 282 us chunks only; [4096,49152] 287 -> 207 us; [2049,100000] 267 -> 239 us.
    resident = false;
    if (rowred && l_min > 1024 && !split_rows) {
      const int e32 = std::max(32, V), e64 = std::max(64, V);
      const bool may_chunk = !colred && !has_transposed;
      int64_t rowv_bytes = 0, full_bytes = 0;
      for (const ExtTensor& e : gp->ext_in) {
        if (e.kind == KIND_ROWV) rowv_bytes += dtype_size(e.dtype);
        if (e.kind == KIND_FULL) full_bytes += dtype_size(e.dtype);
      }
      for (const ExtTensor& e : gp->ext_out)
        if (e.kind == KIND_FULL) full_bytes += dtype_size(e.dtype);
      const bool keep_registers = rowv_bytes < full_bytes;
      if (ecap < e32 && lanes_for(e32) <= 1024 && (opt.wide_level >= 1 || !may_chunk)) ecap = e32, l_min = lanes_for(e32);
      else if (may_chunk && keep_registers && opt.wide_level >= 2 && lanes_for(e64) <= 1024) ecap = e64, l_min = lanes_for(e64);
      else if (may_chunk && keep_registers && opt.wide_level >= 1) resident = true;
    }
    // Row reductions over rows that do not fit the registers of one workgroup: the workgroup walks
    // its row in column chunks, once per stage, recomputing what each stage needs.
    chunked = (l_min > 1024 && rowred && !colred && !has_transposed) || split_rows;
    // Column reductions alone do not need whole rows either: column tiles, each with its own fold.
    // Tiles of 64 lanes x 16 elements, whatever the row length: every tile has its own, small fold (a workgroup's
    // partial is 4 KB, the folds of different tiles run side by side), where one tile as wide as the row makes the last
    // arrivers of the grid fold read 16 x C floats each.  Column sums of f32: [8192,8192] 58 -> 78 % of peak,
    // [16384,4096] 65 -> 69 %, [4096,16384] 71 -> 78 % (tiles of 256 lanes before), narrower rows unchanged.
    col_tiled = colred && !rowred && !has_transposed && (l_min > 1024 || (l_min > 64 && !has_concat));
    // Folds that stream little are bound by latency, above all by the grid-wide fold (~4 us of a 7 us kernel).  Tiles of one
    // 128-byte run let one workgroup, or up to 16 that fold in one level, walk all rows of its columns (beyond 128 trips as many as
    // fill the device, in two levels), and the columns of a tensor fold side by side; several column reductions, and what feeds them, then share a kernel however small it is
    // (worth_fusing).  Whole plans, 256 workgroups and two fold levels -> narrow tiles: column sums + row norms f32 [4765,147]
    // 17.3 -> 8.5 us, [127,1088] 13.4 -> 6.5 us; batch normalisation [1764,512] 21.8 -> 13.6 us, [352,5824] 25.4 -> 11.9 us;
    // LayerNorm backward [318,1145] 17.0 -> 9.7 us.
    //  - Below 16 MB in all (every tensor the kernel touches counts: a group of 8 inputs streams 8 times what its rows hold).
    //  - One [R,C] tensor alone: to 128 MB, in tiles of 32 lanes (64 MB where rows are no multiple of a vector and every tile's
    //    edge shares a line: f32 [500,47169] 18.5 -> 20.9 us, [4096,7681] 24.7 -> 26.0; [4096,3841], 60 MB, 15.8 -> 15.2).
    //    Column sums f32 [4096,1152] 10.3 -> 7.4 us, [8192,2880] 19.6 -> 17.2, [2000,15712] 23.5 -> 21.6, bf16 [8192,5760] 23.3 ->
    //    17.5; batch normalisation [16384,1024] 56.4 -> 52.4.  From 16384 rows on a tile needs many workgroups and the two-level
    //    fold again: 3 % or less on either side for 260 and 512 columns, f32 [24000,1000] 20.1 -> 21.2 us, [65536,500] 94.8 -> 104.6.
    //  - Several, each below 16 MB: to 64 MB, from 128 to 4096 rows.  Sums of 4 inputs f32 [1000,4000] 20.0 -> 12.6 us, [4096,1000] 21.2 -> 19.8;
    //    taller tensors leave the device idle on few tiles, larger ones stream better in wide ones ([16000,255], 62 MB, 16.1 -> 20.7;
    //    8 inputs [16000,100] 14.9 -> 24.6, [4096,1000], 125 MB, 27.2 -> 36.5; bias gradient [8192,2048] 37.6 -> 42.6 us).
    // Their 1024-lane workgroups leave a lane 128 registers: 96 for what a trip's rows, the accumulators and the [1,C] operands
    // take in fp32, the rest for addresses and what is computed.  Sums of 16 bf16 inputs, or 12 of u8, do not fit a single trip.
    int row_tensors = 0;  // [R,C] tensors, and [R,1] operands, which every tile reads again
    narrow_trip_regs = 0;
    narrow_regs = V * (int)gp->col_reduces.size();
    for (const ExtTensor& e : gp->ext_in) {
      row_tensors += e.kind == KIND_FULL || e.kind == KIND_COLV;
      narrow_trip_regs += e.kind == KIND_FULL ? V : e.kind == KIND_COLV ? 1 : 0;
      narrow_regs += e.kind == KIND_ROWV ? V : 0;
    }
    for (const ExtTensor& e : gp->ext_out) row_tensors += e.kind == KIND_FULL;
    const bool narrow_form = opt.narrow_tiles && colred && !rowred && !has_transposed && !has_concat && R > 1 && narrow_trip_regs + narrow_regs <= kNarrowRegs;
    const uint64_t bytes = gp->min_hbm_bytes;
    narrow_lanes = 0;
    // From 16384 rows on tiles of 16 lanes (column sums f32 [65536,38] 9.0 us, 10.1 of 8 lanes; sums + maxima + row norms [40000,38]
    // 11.7 and 12.7), 8 for one fp32 reduction whose rows they fill exactly (batch normalisation [40000,64] 24.5 -> 21.0 us,
    // [20000,64] 22.4 -> 18.7, 21.6 as whole rows).  A plain fold of a tensor that no other kernel reads gains nothing from 16
    // lanes: [30000,100] 8.8 us as whole rows, 9.6 in tiles, [20000,200] 9.2 and 9.6 (after a kernel that read it too, it does:
    // [40000,100] with row norms 22.8 and 20.6).
    if (narrow_form && bytes < (16u << 20)) {
      narrow_lanes = R > 16384 && NV > 8 && !(NV % 8 == 0 && V == 4 && gp->col_reduces.size() == 1) ? 16 : 8;
      if (narrow_lanes == 16 && V == 4 && gp->members.size() == 1 && gp->reads_alone) narrow_lanes = 0;
    } else if (narrow_form && row_tensors == 1 && R <= 16384 && bytes < (C % V ? 64u << 20 : 128u << 20)) narrow_lanes = 32;
    else if (narrow_form && row_tensors > 1 && R >= 128 && R <= 4096 && (int64_t)R * C * max_es < (16 << 20) && bytes < (64u << 20)) narrow_lanes = 8;
    if (narrow_lanes > 0) {
      // Tiles beyond what the device holds at once pay their fixed cost (launch, fold, barriers) in rounds, and rows too few for a
      // wavefront leave lanes idle: less than two rounds of resident lanes (f32 [16,131072] 6.5 -> 3.4 us, [32,122880] 6.7 -> 4.5,
      // [64,122880] 8.3 -> 7.6, [128,122880] 12.8 -> 11.3; but [4,524288], two rounds, 4.4 -> 5.3, [32,245760] 8.1 -> 9.0,
      // [64,245760] 10.6 -> 13.6, [2,1048576], four, 3.7 -> 9.0).  Less than four where 32 lanes a row make workgroups of 256 or 512,
      // several to a compute unit, one streaming while another folds ([8,983040] 8.3 -> 7.0 us, [16,491520] 8.3 -> 7.4; but
      // [16,983040], eight, 11.6 -> 12.8, and workgroups of 128, [4,1966080], 7.5 -> 8.6).
      // Above 16 MB a last round that is more than half empty does not pay either (307 tiles on 256 compute units: f32 [500,39296]
      // 15.4 -> 16.0 us, bf16 [500,78624] 17.1 -> 19.0; 820: bf16 [300,209696] 23.7 -> 25.5; but 410: f32 [300,52416] 13.0 -> 12.1).
      const int64_t tiles = (NV + narrow_lanes - 1) / narrow_lanes;
      const int wg = std::max(64, std::min(1024, narrow_lanes * pow2_ceil(std::min(R, 1024))));
      const int rounds = narrow_lanes == 32 && (wg == 256 || wg == 512) ? 4 : 2;
      if (tiles * wg >= rounds * RES || (bytes >= (16u << 20) && tiles > CUS && tiles % CUS > 0 && tiles % CUS < CUS / 2)) narrow_lanes = 0;
      // (a tile has a workgroup of its own at least: a hint of fewer blocks is kept by the form over whole rows)
      l_hint = std::min(8, l_min);
      const int hinted = hinted_lanes() > 0 ? hinted_lanes() : narrow_lanes;
      if (opt.has_hint && opt.hint.max_workgroups > 0 && opt.hint.max_workgroups < (NV + hinted - 1) / hinted) narrow_lanes = 0;
    }
    narrow_tiles = narrow_lanes > 0;
    col_tiled |= narrow_tiles;
    if (l_min > 1024 && !tileable && !chunked && !col_tiled)
      FS_FAIL(FS_ERR_UNSUPPORTED, "rows of %d columns are too long for one workgroup in a group with %s", C,
              colred ? "row and column reductions" : "transposed outputs");
    if (has_concat && (chunked || col_tiled))
      FS_FAIL(FS_ERR_UNSUPPORTED, "a concat cannot be read by a kernel that walks rows of %d columns in chunks", C);
    if (tileable) l_min = std::min(l_min, 256);
    // transposes: 2-D tiles through LDS, down to rows of 16 elements (a tile of whole narrow rows holds few of them, so it leaves
    // in runs of 16-64 bytes: [65536,256] bf16 85.0 -> 13.9 us as 2-D tiles, f32 93.8 -> 23.7 us; [65536,177] f32 64.5 -> 21.0 us;
    // [65536,64] f32 8.1 -> 7.1 us)
    tiled_transpose = has_transposed && tileable && C >= 16 && R > 1;
    if (split_rows) l_min = 256;
    else if (chunked) l_min = 1024;  // (measured: the largest workgroup keeps the fewest rows in flight, so re-reads hit the caches more often)
    if (!narrow_tiles) l_hint = chunked || col_tiled ? 64 : l_min;
    if (col_tiled) l_min = std::min(narrow_tiles ? narrow_lanes : 64, l_max);
    return FS_OK;
  }

  // lanes per row
  fs_status pick_lanes() {
    L = rowred ? std::min(64, l_max) : std::min(256, l_max);
    // Very narrow rows: a row of at most 32 bytes belongs to one lane (no cross-lane step at all;
    // [4M,3] L2-normalise: 34.8 -> 17.6 us); rows that can only be read element by element (concats
    // with an odd seam) get at least two elements per lane.
    // A row that leaves part of a wavefront's last vector slots empty (768 bf16 columns: 96 vectors
    // on 64 lanes x 2) is better served by fewer lanes that it fills exactly, several rows per
    // wavefront (32 lanes x 3: LayerNorm+GeLU bf16 [32768,768] 24.0 -> 20.9 us).
    // Below a quarter of the slots empty it does not pay (softmax fp32 [32768,640]: 27.7 us on 64 lanes
    // x 3 vectors with 17 % empty, 29.4 us on 32 x 5).
    // How many vectors a lane may take for it: a wavefront's access then covers runs of l x 16 bytes, and what is left of a
    // cache line is fetched again for the lane's next vector.  Two for short runs, three from 512 bytes on, or from 256 bytes on
    // where a vector holds 8 elements and empty slots cost more arithmetic (masked softmax bf16 [22727,264]: 16 x 3 9.4 us, 32 x 2
    // 10.8 us; softmax fp32 [35714,168]: 10.9 against 9.9 us)
    // (softmax fp32 [500000,37], 10 vectors: 2 lanes x 5 122 us, 4 x 3 62 us, 8 x 2 30 us, 16 x 1 31 us; [400000,65]: 4 x 5
    // 107 us, 16 x 2 38 us, 32 x 1 49 us; [200000,161]: 16 x 3 54 us, 32 x 2 45 us; masked softmax bf16 [32768,577]: 32 x 3
    // 22.5 us, 64 x 2 25.7 us).  Runs of whole cache lines (rows of a multiple of 128 bytes, 8 lanes or more) have no such
    // remainder: there the fewest empty slots win (masked softmax bf16 [32768,320]: 16 x 3 12.7 us, 32 x 2 14.9 us).
    // Three on 32 lanes only while rows of 4-element vectors fit the caches: from 64 MB on 64 x 2 streams better (softmax fp32
    // [43024,342] 22.9 -> 21.3 us, [82695,317] 39.4 -> 37.2, residual+LayerNorm fp32 [27212,289] 21.3 -> 20.5, masked softmax fp32
    // [36282,289] 23.5 -> 21.8; below, softmax [20000,289] 9.4 -> 9.5, [5442,289] 4.0 -> 4.5).
    if (rowred && !colred && L > l_min && l_min >= 1) {
      const auto waste = [&](int lanes) { return (int64_t)((NV + lanes - 1) / lanes) * lanes - NV; };
      const bool streams = V == 4 && gp->min_hbm_bytes >= (64u << 20);
      if (waste(L) * 4 >= NV + waste(L))
        for (int l = L / 2; l >= std::max(l_min, 4); l /= 2) {
          const bool whole_lines = (int64_t)C * max_es % 128 == 0 && l >= 8;
          if (whole_lines ? waste(l) < waste(L) : (NV + l - 1) / l <= (l >= (streams ? 64 : 32) || (l >= 16 && V >= 8) ? 3 : 2) && waste(l) <= waste(L)) L = l;
        }
    }
    if (rowred && !colred && (int64_t)C * max_es <= 32) L = 1;
    else if (rowred && !colred && V == 1 && NV >= 4) L = std::min(L, pow2_ceil(NV) / 2);
    // a transposed root leaves as runs of G = WG/L consecutive elements: at least 16 rows per workgroup
    if (has_transposed && !rowred) L = std::min(L, std::max(l_min, 16));
    // looping (column-reduction) kernels want more bytes in flight per lane: 16 elements per lane
    if (colred) L = std::min(L, std::max(1, pow2_ceil((NV * V + 15) / 16)));
    L = std::max(L, l_min);
    if (col_tiled) L = l_min;
    // tile = tt_rows rows (128 bytes of the narrowest transposed output: the length of a run in the
    // transposed tensor) by 1024 / tt_rows lanes x one 16-byte vector; measured best among 14 shapes
    tt_rows = 64;
    if (tiled_transpose) {
      int es = 4;
      for (const ExtTensor& e : gp->ext_out)
        if (e.transposed) es = std::min(es, dtype_size(e.dtype));
      tt_rows = std::max(16, std::min(64, 128 / es));
      L = std::min(1024 / tt_rows, l_max);
      // the tile holds one float per element: 16-element vectors (u8 alone) need narrower tiles to fit the budget
      while (L > 4 && (int64_t)L * V * (tt_rows + 1) * 4 > opt.lds_budget) L /= 2;
      // narrower tiles, down to 64 columns, where a quarter of the tiles' columns would be empty ([65536,139] bf16 14.3 -> 12.3 us,
      // f32 18.5 -> 17.6 us; [9000,130] f32 5.2 -> 3.6 us; 32 columns f32: 19.9 us)
      const auto empty = [&](int lanes) { return (NV + lanes - 1) / lanes * lanes - NV; };
      while (L * V > 64 && empty(L) * 4 >= NV + empty(L) && empty(L / 2) < empty(L)) L /= 2;
      if (tile_hints() && hinted_lanes() > 0) L = hinted_lanes();
    }
    // small problems: more lanes per row until the device has ~8 wavefronts per CU
    // (a row that will be cut into column tiles anyway is not a small problem)
    const bool col_tiles_anyway = tileable && (int64_t)NV * V > (int64_t)L * ecap;
    while ((int64_t)R * L / 64 < 8 * CUS && L < l_max && !(has_transposed && !rowred) && !chunked && !col_tiled && !col_tiles_anyway) L *= 2;
    if (split_rows) L = 256;
    if (hinted_lanes() > 0 && !tiled_transpose && !split_rows) L = hinted_lanes();
    return FS_OK;
  }

  // vectors per lane, column tiles / chunks per row
  fs_status pick_vectors() {
    NVL = (NV + L - 1) / L, CT = 1;
    if (NVL * V > ecap && tileable) {
      NVL = std::max(1, ecap / V);
      CT = (NV + NVL * L - 1) / (NVL * L);
    }
    if (tiled_transpose) {
      NVL = 1;
      // 2-byte elements: two vectors per lane make the tile's rows 512-byte runs like those of f32 tiles; the tile
      // (one float per element) then takes 66.5 KB, which two workgroups per CU still fit -- unless the caller set a budget
      // (bf16 transposes: [32768,8192] 198 -> 182 us, [16384,4096] 49.0 -> 46.9 us; f32 with two vectors: slower; so are
      // bf16 tensors with few tiles either way: [65536,1024] 49.9 -> 51.5 us, [1000,30000] 37.0 -> 38.0 us, [2048,2048])
      int es_in = 4;
      for (const ExtTensor& e : gp->ext_in)
        if (e.kind == KIND_FULL) es_in = std::min(es_in, dtype_size(e.dtype));
      if (es_in == 2 && V == 8 && !opt.lds_budget_given && (int64_t)2 * L * V * (tt_rows + 1) * 4 + 1024 <= device_limits().lds_per_workgroup / 2 &&
          NV >= 16 * L && R >= 4096 && (int64_t)R * C * 2 >= (32ll << 20))
        NVL = 2;
      CT = (NV + NVL * L - 1) / (NVL * L);
    }
    NVLC = 0, RESV = 0;
    if (chunked || col_tiled) {
      NVLC = std::max(1, 16 / V);
      // column tiles: 64 bytes of the narrowest input per lane and trip (bf16: 32 elements), not beyond the row
      // (bf16 column sums of [16384,4096]: 30.5 -> 26.7 us); 32 accumulators per column reduction at most
      if (col_tiled && gp->col_reduces.size() <= 2) NVLC = std::max(1, std::min(std::min(4, 32 / V), (NV + L - 1) / L));
      if (narrow_tiles) NVLC = 1;
      NVL = resident ? std::max(1, (opt.wide_level >= 2 ? 48 : 32) / V) : NVLC;  // (64 resident elements plus a chunk in flight spill)
      RESV = resident ? NVL * L : 0;
      CT = (NV - RESV + NVLC * L - 1) / (NVLC * L);
    }
    return FS_OK;
  }

  // Rows that are no whole cache lines: vectors that begin with the row straddle a line in every access of a wavefront, and a line that is
  // stored in two parts is read again by the memory.  Such rows are held in pieces of whole lines instead (fs_lead_inside), where the
  // lanes of a row need not hold a [1,C] operand or a column's sum (their columns change from row to row), and no order of sums is kept for
  // other kernels of the plan (measure_group).  softmax fp32 [2048,50001] 164.5 -> 154.8 us, [3000,40001] 188.4 -> 182.1,
  // [2048,50000] 155.2 -> 147.5, [1024,65000] 106.3 -> 97.8, [16384,5000] 110.9 -> 103.5, [60000,1025] 87.0 -> 80.6,
  // [1000,5001] 8.1 -> 7.5; masked softmax bf16 [8192,4097] 40.4 -> 32.9, [4000,8001] 37.5 -> 33.7, [20000,801] 18.8 -> 18.3.  16 bytes a lane on fewer
  // lanes in the place of pairs lose (bf16 [16384,577] 11.5 against 12.8).
  // From 32 MB on where rows have 16 KB or more, else from 96 MB on (118 sizes of 10 to 180 MB): below, the ends of the rows cost
  // more than the lines (masked softmax bf16 [5204,1281] 9.6 against 11.0 us, [2600,641] fp32 5.0 and 5.3; softmax [62,20003] 6.1 and 6.3; but
  // [83,20003] bf16 7.4 -> 6.6).  Not for rows of a few lines, all of which the ends touch (softmax fp32 [120000,321] 50.5 against 54.1 us, [60000,385] 31.1 and 31.4,
  // masked softmax bf16 [60000,449] 28.5 and 31.2, [32768,577] 21.2 and 21.1).  A vector more a lane than the row alone needs: fp32 from 256 MB on ([8192,8191] 90.3 -> 86.8, [2048,32767] 101.9 -> 95.3,
  // [65536,1001] 90.3 -> 87.9; at 131 MB [4000,2047] 12.8 -> 13.5; masked softmax bf16 [8192,8191] 72.6 -> 78.4).  Rows that fill a compute unit's
  // registers to the last vector are held in whole vectors, if not in whole lines, where that suffices to ask for them ahead (pick_grid).  Where they are
  // not, whole vectors gain nothing sure: softmax fp32 [700,36862] 41.5 -> 44.3 us, [1500,61438] 151.9 and 152.1, [2048,65533] 216.9 -> 211.4.
  void lead_rows() {
    int min_es = 4;
    bool plain = opt.lead && !several_tiles() && rowred && !colred && !chunked && !resident && !split_rows && !has_transposed && !has_concat && CT == 1 && V >= 2 && L >= 8 && !gp->exchanges;
    for (const auto* list : {&gp->ext_in, &gp->ext_out})
      for (const ExtTensor& e : *list) {
        if (e.kind == KIND_FULL) min_es = std::min(min_es, dtype_size(e.dtype));
        plain &= e.kind != KIND_ROWV;
      }
    for (int m : gp->members) plain &= gp->kind.at(m) != KIND_ROWV;
    if (!plain || C % (128 / min_es) == 0 || (int64_t)C * max_es < 1600 || gp->min_hbm_bytes < ((int64_t)C * max_es >= 16000 ? 32u << 20 : 96u << 20)) return;
    for (int line : {128 / min_es, V}) {
      const int nv = lead_vectors(C, V, line), nvl = (nv + L - 1) / L;
      if (nvl <= NVL + (V == 4 && NVL * V < 32 && gp->min_hbm_bytes >= (256u << 20))) {
        NV = nv, NVL = nvl, lead = line;
        return;
      }
      if (C % V == 0 || L != 1024 || NVL * V < 32 || R <= CUS || R > 2 * CUS) return;
    }
  }

  // The groups of a chain take the lanes a row that the widest one has.  In the others half of them or more would compute on what is no
  // column, and a wavefront alone on its SIMD issues an instruction every four cycles, whatever the lanes do: rows of one vector a lane
  // are spread over up to four times their lanes, an element or two to each.  (fs_gather keeps the order of their sums.)  Random DAG of 200
  // ops, whose chain of [512,128], [512,64] and [512,256] takes 64 lanes: [512,256] 19.5 -> 18.7 us, [1911,384] 45.4 -> 44.3, [64,128] 14.2 -> 13.8.
  int spread_rows() {
    int spread = 1;
    while (!lead && opt.fill_lanes && !colred && !has_concat && !tiled_transpose && !chunked && NVL == 1 && CT == 1 && spread < 4 && V % 2 == 0 && C % V == 0 && 2 * NV <= L) V /= 2, NV *= 2, spread *= 2;
    return spread;
  }

  // Wide rows of kernels that reduce rows and columns, one workgroup of 512 lanes to a compute unit (plan_lds): such a workgroup asks
  // for the rows of its next trip before it works on those it has.  Rows of whole vectors and trips of whole groups of rows: a branch
  // around the loads or stores would have the compiler wait for all of them.  Where this takes 512 lanes in the place of 1024, from
  // 12 trips on.  That is not where the two measure the same: fewer trips gain as well (LayerNorm backward [3000,4096] 40.2 -> 34.6 us,
  // [2048,8192] 56.9 -> 47.0), and so would row counts that leave a partial trip ([8191,4096] takes 82 us, [8192,4096] 74).
  bool columns_ahead() const {
    const int64_t trips = R / std::max(1, 512 / L);
    return opt.ahead && rowred && colred && !col_tiled && !has_transposed && !has_concat && CT == 1 && C >= 2048 && C % V == 0 && L <= 512 && whole_lanes && row_inputs > 0 &&
           R % (512 / L) == 0 && (L < 256 ? trips > CUS : trips >= 12 * (int64_t)CUS);
  }

  // workgroup size; whether workgroups loop with their [1,C] operands staged once
  fs_status pick_workgroup() {
    for (const ExtTensor& e : gp->ext_in) {
      row_inputs += e.kind == KIND_FULL;
      whole_lanes &= e.kind != KIND_FULL || V * dtype_size(e.dtype) == 16;
    }
    int flipped = 0;  // values that leave transposed
    for (const ExtTensor& e : gp->ext_out) flipped += e.transposed;
    const int64_t total_waves = std::max<int64_t>(1, (int64_t)R * CT * L / 64);
    if (narrow_tiles) {
      WG = std::max(64, std::min(1024, L * pow2_ceil(std::min(R, 1024))));
    } else if (col_tiled) {
      WG = std::max(64, L);
      for (int w = 512; w >= 128; w /= 2)
        if (w >= L && (int64_t)R * L / w >= 8) {
          WG = w;
          break;
        }
    } else if (colred) {
      // large workgroups (few partials, many rows per trip) as long as every CU still gets a workgroup
      // and the in-workgroup fold area (one row of C floats per wavefront or row-group) fits the budget
      WG = std::max(64, L);
      for (int w = 512; w >= 128; w /= 2)
        if (w >= L && (int64_t)R * L / w >= CUS) {
          WG = w;
          break;
        }
      // rows across several wavefronts: 16 wavefronts per CU.  8 where rows that no whole vectors fill leave the kernel too, 20 elements
      // to a lane or 512 lanes to a row: such kernels are short of registers at 16 (LayerNorm backward [2500,4101] 58.7 -> 51.3 us, [6000,4801] 108.5 ->
      // 92.5, [4000,6201] 101.5 -> 90.9, [3000,8191] 94.1 -> 89.8; with 16 elements on 256 lanes, [5000,3501], 57.2 against 61.6)
      bool writes = false;
      for (const ExtTensor& e : gp->ext_out) writes |= e.kind == KIND_FULL;
      if (rowred && L >= 256) WG = std::max(WG, columns_ahead() || (C % V != 0 && writes && (NVL * V > 16 || L >= 512)) ? 512 : std::min(1024, 4 * L));
    }
    // Four rows to a workgroup, where there is LDS for the tile that takes them, rather than two whose transposed values leave one by one:
    // where there are several of them.  Random DAG of 200 ops [700,384] 31.9 -> 25.4 us, [1000,384] 36.5 -> 31.2, [1911,384] 50.0 -> 45.6, [128,384] 21.3 ->
    // 19.4; 8 rows 29.3, 34.8, 44.5, 26.2.  With one such output fewer workgroups cost more ([1000,128] 18.3 against 20.8).  Not while groups are
    // formed: what would be fused for it costs more than it saves ([1911,384] 59.5).
    else if (opt.grouped && rowred && flipped >= 2 && L >= 128 && L <= 256 && (int64_t)C * 20 + 4096 <= opt.lds_budget) WG = 4 * L;
    else if (total_waves > 4 * CUS || has_transposed) WG = std::max(256, L);
    else WG = std::max(64, L);
    // Rows with [1,C] operands, above all operands that outweigh the row's own traffic (LayerNorm with
    // gamma, beta and a bias over bf16 rows: 12 bytes per column against 4).  Re-reading the operands for every row, or for
    // every few rows of a one-trip workgroup, costs L2 bandwidth; keeping them in registers costs
    // occupancy (48 of 84 registers).  When they fit the LDS budget and there is work for more than
    // two rounds of resident workgroups, the workgroups loop instead, 32 wavefronts per CU, and stage
    // the operands in LDS once, before the loop.  LayerNorm+GeLU bf16 [8192,4096]: 35.3 us re-reading,
    // 31.2 us from registers, 27.6 us staged; [16384,2048]: 29.3 -> 26.5 us; [16384,1024]: 14.7 ->
    // 13.1 us (one trip: staged once per 4 rows); no gain without such operands (softmax: 3-7 % slower),
    // nor for one-wavefront rows with fewer than 16 elements per lane or a half-empty last vector
    // ([16384,512]: 9.2 -> 9.7 us, [32768,768]: 22.6 -> 24.1 us), which keep the one-trip form.
    staged_loop = false;
    if (rowred && !colred && !chunked && !has_transposed && CT == 1 && R > 1) {
      int64_t rowv_bytes = 0, full_bytes = 0;
      int n_rowv_in = 0;
      for (const ExtTensor& e : gp->ext_in) {  // bytes per column
        if (e.kind == KIND_ROWV) rowv_bytes += dtype_size(e.dtype), ++n_rowv_in;
        if (e.kind == KIND_FULL) full_bytes += dtype_size(e.dtype);
      }
      for (const ExtTensor& e : gp->ext_out)
        if (e.kind == KIND_FULL) full_bytes += dtype_size(e.dtype);
      const int wg = L >= 128 ? std::min(1024, 4 * L) : std::max(256, std::min(1024, 16 * L));  // 4 rows, or 16 one-wavefront rows, per trip
      // (one-wavefront rows: beyond ~8 rounds of resident workgroups the one-trip form catches up and
      // passes: [65536,1024] 48.9 against 49.5 us, [262144,1024] 203 against 210 us)
      const bool full_slices = NVL * V >= 16 && (int64_t)NVL * L == NV && (int64_t)R * L <= 8 * RES;
      // rows across several wavefronts gain with any [1,C] operand (RMSNorm bf16 [8192,4096]: 24.5 ->
      // 23.6 us, residual+LayerNorm: 50.5 -> 45.8 us); one-wavefront rows only with heavy ones
      // (up to ~4 rounds of work: at [32768,2048] the one-trip form is 2-5 % faster again)
      const bool heavy = rowv_bytes * 2 >= full_bytes * 3;
      // from two rounds of resident workgroups on; from one round where heavy operands meet rows of one or two wavefronts
      // (LayerNorm+GeLU bf16 [8192,1024]: 9.0 -> 8.0 us, [12288,1024]: 11.7 -> 10.6 us, [6000,2048]: 12.4 -> 10.3 us; rows over
      // four wavefronts and light operands lose there: [2048,4096] 9.9 -> 10.6 us, RMSNorm [1024,8192] 6.7 -> 7.7 us)
      const int rounds = heavy && L <= 128 ? 1 : 2;
      const bool pays = L >= 128 ? heavy || (n_rowv_in > 0 && (int64_t)R * L <= 4 * RES) : full_slices && heavy;
      if (pays && (int64_t)n_rowv_in * NVL * L * V * 4 + 1024 <= opt.lds_budget && (int64_t)R * L / wg >= rounds * (RES / wg)) {
        staged_loop = true;
        WG = wg;
      }
    }
    if (chunked) WG = L;  // one row per workgroup
    if (tiled_transpose) WG = std::max(64, std::min(1024, L * std::min(tt_rows, std::max(4, pow2_ceil(std::min(R, 1024))))));
    if (opt.has_hint && opt.hint.wg_threads > 0 && !chunked && (!tiled_transpose || tile_hints())) {
      const int h = opt.hint.wg_threads;
      if (h % 64 == 0 && h % L == 0 && h <= 1024) WG = h;  // (whole rows: lanes left over would share another row group's slots)
    }
    return FS_OK;
  }

  // the schedule record, row segments of split rows, loop trips
  fs_status fill_schedule() {
    s.V = V;
    s.NV = NV;
    s.L = L;
    s.NVL = NVL;
    s.CT = CT;
    s.E = s.NVL * V;
    s.WG = WG;
    s.G = WG / L;
    s.shares_lines = C % V != 0 || in_pairs;
    s.lead = lead;
    s.ragged = !lead && (C % V != 0 || (!resident && (int64_t)CT * NVL * L != NV));
    s.resident = resident;
    s.NVLC = NVLC;
    s.RESV = RESV;
    s.ragged_chunks = chunked && ((int64_t)RESV + (int64_t)CT * NVLC * L != NV || C % V != 0);
    s.chunked = chunked;
    s.col_tiled = col_tiled;
    s.narrow_tiles = narrow_tiles;
    s.tiled_transpose = tiled_transpose;
    // Bands whose rows are 4 KB runs of the narrowest input (8 tiles of f32, 16 of bf16), twice that when the tensor has
    // so few row tiles that a band would not fill the device.  Against plain order, f32: [8192,8192] 60 -> 75 % of peak,
    // [1024,65536] 51 -> 72 %, [8192,28672] 58 -> 70 %, [300,100000] 34 -> 63 %; bf16: [32768,8192] 56 -> 66 %,
    // [1000,30000] 30 -> 46 %; never slower on 24 shapes.  (Bands of 2 or 4 tiles are slower than none; the best
    // width varies by a few per cent with the row pitch, [16384,16384] f32: 66 % with 8, 61 % with 16, 68 % with 24.)
    s.tt_col_band = 0;
    if (tiled_transpose) {
      int es = 4;
      for (const ExtTensor& e : gp->ext_in)
        if (e.kind == KIND_FULL) es = std::min(es, dtype_size(e.dtype));
      const int row_tiles = (R + s.G - 1) / s.G;
      int band = std::max(1, 4096 / (NVL * L * V * es));
      if (row_tiles <= 32) band *= 2;
      if (CT > band) s.tt_col_band = band;
    }
    s.split_rows = split_rows;
    s.min_waves = opt.min_waves;
    s.few_long_rows = few_long_rows;
    s.S = 1;
    s.CPS = CT;
    if (split_rows) {  // at least 2 chunks per workgroup, about `target` workgroups in all
      const int target = opt.has_hint && opt.hint.max_workgroups > 0 ? opt.hint.max_workgroups : 512;
      s.S = std::max(1, std::min((CT + 1) / 2, std::max(1, target / R)));
      s.CPS = (CT + s.S - 1) / s.S;
      s.S = (CT + s.CPS - 1) / s.CPS;  // no empty segment
    }
    s.n_iters = split_rows ? R * s.S : chunked ? R : col_tiled ? (R + s.G - 1) / s.G : tiled_transpose ? (int)((int64_t)CT * ((R + s.G - 1) / s.G))
                                                                               : (int)(((int64_t)R * CT + s.G - 1) / s.G);
    return FS_OK;
  }

  // workgroups launched, row tiles per trip, fold fan-in
  fs_status pick_grid() {
    // Streaming groups launch one workgroup per row tile: the hardware hands tiles out in memory
    // order and a fresh wavefront issues its loads at once, which measures faster on this device
    // than persistent workgroups looping with a grid stride.  Column reductions keep a bounded
    // grid because every workgroup leaves a partial to fold.
    int cap = colred ? CUS : (1 << 30);
    // Exception: [1,C] operands that cannot be shared through LDS (fewer than 4 rows per workgroup)
    // are read again from L2 for every row of a one-shot grid.  When those reads outweigh the row's
    // own traffic (LayerNorm with gamma, beta and a bias over rows of 4096+ elements: 12 bytes per
    // column against 4), the workgroups loop instead, 16 wavefronts per CU, and keep their slices of
    // the operands in registers (measured on [8192,4096] bf16: 35.3 -> 29.4 us).
    if (staged_loop && s.G >= 2) {
      cap = std::max(CUS, (int)(RES / WG));
    } else if (!colred && !chunked && CT == 1 && s.G < 4 && R > 1) {
      int64_t rowv_bytes = 0, full_bytes = 0;
      for (const ExtTensor& e : gp->ext_in) {  // bytes per column
        if (e.kind == KIND_ROWV) rowv_bytes += dtype_size(e.dtype);
        if (e.kind == KIND_FULL) full_bytes += dtype_size(e.dtype);
      }
      for (const ExtTensor& e : gp->ext_out)
        if (e.kind == KIND_FULL) full_bytes += dtype_size(e.dtype);
      if (rowv_bytes * 2 >= full_bytes * 3) cap = std::max(CUS, (int)(RES / 2 / WG));
    }
    // Rows that fill a compute unit's registers, one workgroup to a unit: loads, arithmetic and stores of a row would follow each
    // other.  One workgroup per unit stays instead and asks for its next row, mostly through LDS, before it works on a row (loads
    // asked for after the stores wait for them: 14-20 % slower).  softmax fp32 [1024,65536] 111.1 -> 104.3 us, [2048,50000] 160.0 -> 153.3,
    // [2048,32768] 97.1 -> 94.3, [300,65000] 53.1 -> 47.1, [400,50000] 35.2 -> 32.5; a copy in such rows takes 144 us for the second.
    // Below 32 elements per lane two workgroups share a unit, which is better ([4096,20000] 108.8 against 115.0).  Rows that are no
    // whole vectors: up to two a workgroup, as test_which_long_rows_are_asked_for_ahead has it.  In pieces of whole lines (lead_rows) a lane asks for 16 aligned
    // bytes, and more rows would gain too ([2048,50001] 154.8 us, 146.5 ahead, [3000,40001] 182.1 and 171.1).  Those whose pieces would need a vector more a
    // lane cross to LDS in 4-byte pieces, which eats the gain ([2048,33001] 104.7 against 106.3) but for a few rows ([500,53247] 41.0 us, 46.4 without, [400,40959]
    // 24.7 and 28.6, [512,65535] 55.6 and 59.0; a vector more 41.2, 26.5 and 62.4).  Only for kernels that write rows: all that was measured and
    // checked did.
    bool rowv = false, writes = false;
    for (const ExtTensor& e : gp->ext_in) rowv |= e.kind == KIND_ROWV;
    for (const ExtTensor& e : gp->ext_out) writes |= e.kind == KIND_FULL;
    s.ahead = opt.ahead && !several_tiles() && writes && rowred && !colred && !chunked && !resident && !has_transposed && !has_concat && CT == 1 && s.G == 1 && WG == 1024 && s.E >= 32 && row_inputs == 1 && !rowv &&
              whole_lanes && R > CUS && (C % V == 0 || (R <= 2 * CUS && (lead || max_es == 4)));
    if (s.ahead) {
      const int lds = opt.lds_budget_given ? opt.lds_budget : device_limits().lds_per_workgroup;
      s.ahead_lds = std::min(C / (L * V), (lds - 2048) / (WG * 16));
      s.ahead = s.ahead_lds >= 1 && NVL - s.ahead_lds <= 8;
      if (s.ahead) cap = CUS;
    }
    if (opt.has_hint && opt.hint.max_workgroups > 0) cap = opt.hint.max_workgroups;
    cap = std::min(cap, (int)(0x7fffffff / WG));  // a launch holds fewer than 2^31 lanes: beyond that the workgroups loop
    s.grid = std::max(1, std::min(s.n_iters, cap));
    // workload 2 (2 trips): 13.5 -> 13.0 us; LayerNorm+GeLU bf16 [12288,1024]: 10.7 -> 10.2 us; 4 trips: +0.4 %, 8 trips: -0.8 %;
    // rows over several wavefronts lose 3-16 % ([6000,2048]: 10.5 -> 12.3 us)
    s.rotate_loop = staged_loop && L <= 64 && s.grid < s.n_iters && s.n_iters <= 4 * (int64_t)s.grid;
    s.RB = s.grid;
    if (split_rows) {
      s.grid = R * s.S;
      s.RB = s.S;
    }
    if (col_tiled) {  // RB workgroups per column tile, about `cap` workgroups in all
      s.RB = std::max(1, std::min(s.n_iters, std::max(1, cap / CT)));
      // Narrow tiles: a workgroup takes up to 4 trips, whose loads it keeps in flight together, and up to 8 where that keeps the
      // fold at one level of 16.  Four trips of one workgroup beat two workgroups of two, which have partials to exchange: column
      // sums f32 [512,1000] 3.1 against 4.6 us, [400,4000] 3.1 against 4.9; sum, max and sum of squares bf16 [512,2000] 7.9
      // against 9.7; batch normalisation [512,1000] 9.4 against 12.3 us.
      if (narrow_tiles && !(opt.has_hint && opt.hint.max_workgroups > 0)) {
        const int want = (s.n_iters + 3) / 4;
        if (want <= 32) s.RB = std::min(s.RB, std::min(want, 16));
      }
      s.grid = s.RB * CT;
      if (tiles_share_lines(*gp)) s.xcd_rows = 8;
    }
    // Looping kernels that only fold columns have almost no arithmetic per trip: their rate is set by
    // the bytes in flight, and two row tiles per trip measured 13 % faster (28.1 -> 24.5 us on
    // [65536,512]).  With a row reduction in the body one tile per trip is the faster form.
    s.U = (colred && !rowred && s.grid < s.n_iters && CT == 1) ? 2 : 1;
    if (narrow_tiles) {  // all loads of a few trips in flight, as far as they fit the registers
      // (sum of 4 bf16 inputs [2000,512]: 4 trips 9.2 us, 2 trips 6.5; of 8 inputs [1000,4000]: 2 trips 23.6, 1 trip 17.8)
      const int trips = (s.n_iters + s.RB - 1) / s.RB;
      s.U = trips >= 4 ? 4 : trips >= 2 ? 2 : 1;
      while (s.U > 1 && s.U * narrow_trip_regs + narrow_regs > kNarrowRegs) s.U /= 2;
    }
    if (opt.has_hint && opt.hint.tiles_per_trip >= 1 && opt.hint.tiles_per_trip <= 4) s.U = opt.hint.tiles_per_trip;
    if (has_concat || tiled_transpose) s.U = 1;
    // two fold levels at most: the smallest fan-in whose square covers the grid (one level for narrow tiles of up to 16 workgroups)
    // (64 workgroups per fold: 16 measured 9 % faster than 8 on column sums of [16384,4096], 44.6 against 48.8 us)
    s.fan_in = s.RB <= 16 && narrow_tiles ? 16 : s.RB <= 32 ? 8 : s.RB <= 256 ? 16 : 32;
    // One-trip grids whose workgroups share cache lines with their neighbours: in a transposed tensor, into which a workgroup writes a few rows
    // of a line (8 workgroups of 4 fp32 rows fill one), and at the ends of rows that are no whole lines.  Placed in turn on the XCDs, each of two
    // L2s moves such a line; now 8 or 16 neighbours run on one XCD.  Random DAGs of 200 ops [512,256] 21.4 -> 20.4 us, [700,384] 36.0 -> 31.4, [1500,256]
    // 31.2 -> 27.6 (4: 28.0, 16: 28.1); masked softmax bf16 [16384,577] 11.26 -> 11.12, [32768,129] 7.6 -> 7.1, softmax fp32 [2048,50001] 168.7 -> 164.4 (4 and 8:
    // three fifths of that), elementwise of 6 tensors [16384,1001] 67.8 -> 66.2, LayerNorm+GeLU bf16 [8000,1021] 7.1 -> 6.7.  Rows of whole lines have nothing to gain
    // ([16384,1024] 64.3 and 64.3; an eighth of all rows to an XCD, which meets the same channels, 67.9).
    if (!has_concat && !tiled_transpose && !colred && !chunked && CT == 1 && s.U == 1 && s.grid == s.n_iters) {
      bool shared = false;
      for (const auto* list : {&gp->ext_in, &gp->ext_out})
        for (const ExtTensor& e : *list) shared |= e.kind == KIND_FULL && !e.transposed && (int64_t)s.G * C * dtype_size(e.dtype) % 128 != 0;
      s.xcd_rows = has_transposed ? 8 : shared ? 16 : 0;
    }
    // (folds of columns, too, whatever their trips: row softmax numerators, transposed twice, with row and column sums fp32 [4100,700] 21.9 -> 19.3 us,
    // [3000,1500] 30.4 -> 25.5, [9000,400] 22.0 -> 20.1, [2048,1024] 15.4 -> 14.7; rows of a power of two in number and few columns lose 1 to 3 %, [4096,512]
    // 13.0 -> 13.4, [16384,256] 17.9 -> 18.1)
    if (has_transposed && rowred && colred && !tiled_transpose && !chunked && CT == 1 && s.U == 1) s.xcd_rows = 8;
    // (one row to a workgroup that stays: 32 neighbours; few rows leave XCDs idle in the last trip then, 16.  softmax fp32 [1024,65000] 100.8 -> 97.8 us,
    // [400,50001] 30.7 -> 30.5, 34.8 with 32.  Not where every other row begins with a line: test_which_rows_are_placed_by_xcd has [2048,50000] in plain
    // order, 147.5 us, 145.5 with 32)
    if (s.ahead && s.lead && (int64_t)C * max_es % 64 != 0) s.xcd_rows = R >= 4 * CUS ? 32 : 16;
    return FS_OK;
  }

  // LDS plan of the kernel
  fs_status plan_lds() {
    // LDS plan (Section 5.1).  Size requirements: cross-wave row-reduction partials (the "direct
    // allocation" for a non-root Reduce) and the column-partial fold area.  Space sharing: all row
    // reductions of the kernel reuse one ping-pong pair of slots instead of one buffer each (the
    // Reduce.2-reuses-Reduce.1 case of Section 5.1.3); the column fold area is shared by all column
    // reductions in turn.
    // Space sharing by lifetime (the idea of Section 5.1.3 applied to the kernel's two phases): what
    // the row loop uses (transpose tile, staged [1,C] operands) is dead when the epilogue folds the
    // column partials, so both live in one pool of max(loop bytes, fold bytes).
    int fixed = 0, loop_bytes = 0, fold_bytes = 0;
    if (rowred && L > 64) fixed += 2 * s.G * (L / 64) * gp->max_batched_reduces * 4;
    if (split_rows) fixed += 16 + (int)gp->row_reduces.size() * 4;
    // Columns one workgroup folds: its tile, or the row rounded up to 16-byte chunks, one chunk of every reduction per lane and
    // round.  Not where that needs another round for less than half of a workgroup of 512 lanes or less that only reads: there the
    // row as it is, in the chunks that divide it (column sums and maxima + row norms f32 [14396,1101] 26.3 us rounded, 23.3 as it
    // is, [10000,2101] 38.8 and 35.8).  With one round or a full last one the rounded row is faster ([14396,1001] 18.7 and 21.5,
    // [12000,1801] 32.7 and 35.1), with a lane or two in the last one ([12000,1025] 21.7 and 22.9), in larger workgroups
    // ([2500,4501] 30.0 and 35.0), and beside [R,C] outputs (LayerNorm backward [9000,1450] 41.6 and 43.2).
    s.fold_width = col_tiled ? NVL * L * V : C;
    if (!col_tiled && C % 4 != 0) {
      const int64_t chunks = (int64_t)gp->col_reduces.size() * ((C + 3) / 4);
      const int last = (int)(chunks % WG);
      bool writes = false;
      for (const ExtTensor& e : gp->ext_out) writes |= e.kind == KIND_FULL;
      if (chunks <= WG || last < 16 || last >= WG / 2 || WG > 512 || writes) s.fold_width = (C + 3) / 4 * 4;
    }
    const int fold_width = s.fold_width;
    s.fold_piece = fold_width;
    s.meet = 0;
    if (colred) {
      // the fold area takes at most half of the budget: wide rows pass through it in pieces
      fixed += 16;
      const int fold_rows = L < 64 ? WG / 64 : s.G;
      const int piece_cap = std::max(8, (opt.lds_budget / 2 / (fold_rows * 4)) / 8 * 8);
      if (fold_width > piece_cap) s.fold_piece = piece_cap;
      fold_bytes = fold_rows * s.fold_piece * 4;
    }
    auto total = [&]() { return fixed + std::max(loop_bytes, fold_bytes); };
    // [1,C] inputs shared by all rows of a workgroup are staged in LDS by the whole workgroup (once,
    // before the loop, when the workgroup loops) when several rows share them and the budget allows
    int n_rowv = 0;
    for (const ExtTensor& e : gp->ext_in) n_rowv += e.kind == KIND_ROWV;
    s.stage_rowv = false;
    s.tile_transpose = false;
    const int tile_bytes = (tiled_transpose ? NVL * L * V : C) * (s.G + 1) * 4;
    // (the wider tiles of 2-byte transposes may pass the default budget: half of what a CU has, so that two workgroups fit)
    const int tile_cap = tiled_transpose && NVL == 2 ? device_limits().lds_per_workgroup / 2 : opt.lds_budget;
    if (has_transposed && (CT == 1 || tiled_transpose) && s.G >= 4 && fixed + std::max(loop_bytes + tile_bytes, fold_bytes) <= tile_cap) {
      s.tile_transpose = true;
      loop_bytes += tile_bytes;
    }
    const int slot_bytes = s.NVL * s.L * V * 4;
    if (n_rowv > 0 && CT == 1 && (s.G >= 4 || (staged_loop && s.G >= 2)) && R > 1 &&
        fixed + std::max(loop_bytes + n_rowv * slot_bytes, fold_bytes) <= opt.lds_budget) {
      s.stage_rowv = true;
      loop_bytes += n_rowv * slot_bytes;
    }
    // Partials of 16 KB or more from every compute unit: where a tree's last workgroups read 16 of them each, twice, on one unit, all
    // workgroups meet and fold a slice of the columns each.  LayerNorm backward fp32 [4096,8192] 102.7 -> 93.5 us, [5000,3000] 54.4 ->
    // 47.2, [8192,4096] 85.9 -> 82.3, [16384,2048] 80.3 and 80.2; moments bf16 [8192,8192] 69.5 -> 57.7.  To meet takes 2 us more than
    // to pass two tickets, which smaller partials do not return: [16384,1024] 39.6 against 41.1, moments [65536,512] 26.5 against 28.5.  Beyond 2048
    // columns in all a lane of the tree's last workgroup folds a second chunk, and kernels of less than 52 MB are short enough to notice: column sums + row
    // norms [4096,1100] 14.0 -> 12.6 us, [4000,2000] 18.8 -> 16.8, [8192,1536] 18.4 -> 16.9, with a maximum and a mean [4096,1100] 14.6 -> 12.4, [8192,1200] 19.7 ->
    // 17.7, LayerNorm backward [2100,1300] 18.5 and 18.6; above, the tree is as good or better: column sums + row norms [30000,1100] 28.1 and 28.4, LayerNorm backward
    // [8000,1200] 28.3 and 29.2, [16384,1100] 45.2 and 46.4, three folds [20000,1024] 35.6 and 37.1, [8192,1000] 22.1 and 23.3 (but [2500,1900] 23.8 and 23.0).
    const int64_t fold_columns = (int64_t)gp->col_reduces.size() * fold_width;
    if (opt.meet && colred && !col_tiled && s.RB > s.fan_in && s.RB <= CUS && fold_columns > 2048 && (fold_columns >= 4096 || gp->min_hbm_bytes < 52000000)) {
      const int FV = fold_vector(fold_width), chunks = (int)gp->col_reduces.size() * (fold_width / FV);
      const int SC = std::max(16 / FV, std::min(64, pow2_ceil((chunks + s.RB - 1) / s.RB))), meet_bytes = WG / 64 * SC * FV * 4;
      if (fixed + 32 + std::max({loop_bytes, fold_bytes, meet_bytes}) <= opt.lds_budget) {
        s.meet = SC;
        fixed += 32;  // (who has left)
        fold_bytes = std::max(fold_bytes, meet_bytes);
        gp->wait_ticks = wait_ticks(10000);
      }
    }
    // Rows asked for ahead in kernels that reduce rows and columns (columns_ahead): without that one workgroup to a compute unit has
    // few loads in flight while it works on its rows.  Through LDS as far as 40000 bytes go, whose place the column fold takes at the
    // end, the rest to registers (all of it through LDS was no faster).  8 wavefronts, which have the registers, instead of 16, whose
    // trips come in larger bursts.  LayerNorm backward fp32 [8192,4096] 82.6 -> 74.2 us (16 wavefronts: 80.9), [4096,8192] 94.2 ->
    // 78.7 (85.8), [12288,4096] 116.4 -> 107.3 (116.8), [8192,8192] 166.9 -> 147.0 (153.6), [5000,3000] 47.2 -> 43.1, [16384,2048] 81.2 -> 74.2; moments bf16
    // [16384,4096] 55.1 -> 48.4, [16384,2048] 34.2 -> 29.3.  Rows of up to 1024 columns, many to a workgroup, lose (moments [65536,1024] 45.3
    // against 54.3, LayerNorm backward [16384,1024] 39.3 and 39.6).
    if (columns_ahead() && WG == 512 && s.U == 1 && s.grid < s.n_iters) {
      const int most = std::min(opt.lds_budget, 40000), each = row_inputs * WG * 16, fold_rows = L < 64 ? WG / 64 : s.G;
      const int JL = std::min({NVL, C / (L * V), (most - fixed - loop_bytes - 256) / each}), piece = JL * each / (fold_rows * 4) / 8 * 8;
      if (JL > 0) {
        s.ahead = true;
        s.ahead_lds = JL;
        s.fold_piece = std::min(fold_width, piece);
        s.lds_bytes = s.lds_planned = fixed + loop_bytes + JL * each;
        s.stage_avail = 0;
        return FS_OK;
      }
    }
    const int lds = total();
    s.lds_bytes = s.lds_planned = lds;
    if (lds > (s.tile_transpose ? tile_cap : opt.lds_budget))
      FS_FAIL(FS_ERR_LDS_BUDGET, "group needs %d bytes of LDS, budget is %d", lds, opt.lds_budget);
    // Rows walked in chunks: what is left of the workgroup's LDS may hold the head of the row in its input dtype
    // (one 1024-lane workgroup per compute unit runs such a kernel, so it may take all a workgroup is allowed
    // unless the caller set a budget); code generation decides which inputs are worth it.
    s.stage_avail = 0;
    if (s.ahead && !colred) s.lds_bytes = s.lds_planned = lds + row_inputs * s.ahead_lds * WG * 16;  // (a workgroup has its compute unit to itself, like those below)
    if (chunked && !split_rows) {
      const int cap = opt.lds_budget_given ? opt.lds_budget : device_limits().lds_per_workgroup;
      s.stage_avail = std::max(0, cap - lds - 512);
    }
    return FS_OK;
  }

  // workspace scratch of grid-wide folds
  fs_status plan_scratch() {
    // grid-wide fold scratch
    gp->n_tickets = 0;
    gp->part_bytes = 0;
    s.part_stride_floats = 0;
    s.ticket_stride = 0;
    if (split_rows) {  // per row: S partials of one float per reduction
      const size_t k = gp->row_reduces.size();
      int n = s.S;
      while (n > 1) {
        s.part_stride_floats += (size_t)n * k;
        n = (n + s.fan_in - 1) / s.fan_in;
        s.ticket_stride += n;
      }
      gp->n_tickets = s.ticket_stride * R;
      gp->part_bytes = s.part_stride_floats * R * 4;
    }
    if (colred) {
      const size_t kc = gp->col_reduces.size() * (size_t)s.fold_width;
      int n = s.RB;
      while (n > 1) {
        s.part_stride_floats += (size_t)n * kc;
        n = (n + s.fan_in - 1) / s.fan_in;
        s.ticket_stride += n;
        if (s.meet) {  // one level of partials; counters in cache lines of their own, and the doors
          s.ticket_stride = 32 * (1 + (s.RB + 15) / 16) + s.RB;
          break;
        }
      }
      const int tiles = col_tiled ? CT : 1;
      gp->n_tickets = s.ticket_stride * tiles;
      gp->part_bytes = s.part_stride_floats * tiles * 4;
    }
    return FS_OK;
  }

  fs_status run() {
    fs_status st;
    if ((st = measure_group()) != FS_OK) return st;
    if ((st = pick_row_form()) != FS_OK) return st;
    if ((st = pick_lanes()) != FS_OK) return st;
    if ((st = pick_vectors()) != FS_OK) return st;
    if ((st = pick_vector_width()) != FS_OK) return st;
    lead_rows();
    s.spread = spread_rows();
    if ((st = pick_workgroup()) != FS_OK) return st;
    if ((st = fill_schedule()) != FS_OK) return st;
    if ((st = pick_grid()) != FS_OK) return st;
    if ((st = plan_lds()) != FS_OK) return st;
    return plan_scratch();
  }
};
}  // namespace

static fs_status choose_schedule(const Graph& g, const PlanOptions& opt, GroupPlan* gp) { return Scheduler(g, opt, gp).run(); }

fs_status analyse_group(const Graph& g, const std::vector<int>& members, const std::vector<int>& /*group_of*/,
                        int self_group, const PlanOptions& opt, GroupPlan* out) {
  GroupPlan& gp = *out;
  gp = GroupPlan();
  gp.members = members;
  std::sort(gp.members.begin(), gp.members.end());
  Analyser a(g, gp);
  for (int m : gp.members) a.in_set[m] = 1;

  // Orientation of every member.  A transpose inside a group moves no data: it flips the flag,
  // and everything downstream is computed in the producer's register layout (the paper inlines
  // such shape modulation by thread composition, Section 4.3).  Only a value that LEAVES the
  // kernel in the flipped orientation is stored transposed.
  std::map<int, bool>& tf = gp.tflag;
  for (int m : gp.members) {
    const fs_node& n = g.nodes[m];
    bool t = n.opcode == FS_TRANSPOSE;  // operands outside the group are read as they lie in memory
    for (int k = 0; k < n.num_in; ++k) {
      const int src = a.source_of(n.in[k]);
      if (a.in_set[src]) {
        t = (n.opcode == FS_TRANSPOSE) ? !tf[src] : tf[src];
        break;
      }
    }
    tf[m] = t;
  }
  // work space: the largest extents seen, every shape taken in its orientation
  int R = 1, C = 1;
  for (int m : gp.members) {
    const fs_node& n = g.nodes[m];
    const bool t = tf[m], t_op = n.opcode == FS_TRANSPOSE ? !t : t;
    R = std::max(R, t ? n.cols : n.rows), C = std::max(C, t ? n.rows : n.cols);
    for (int k = 0; k < n.num_in; ++k) {
      if (g.flat_in[m][k]) continue;  // read as an element sequence under this node's own shape: its label says nothing here
      const fs_node& o = g.nodes[n.in[k]];
      R = std::max(R, t_op ? o.cols : o.rows), C = std::max(C, t_op ? o.rows : o.cols);
    }
  }
  a.R = gp.R = R;
  a.C = gp.C = C;

  auto is_reduce = [&](int id) { return g.nodes[id].opcode == FS_REDUCE_ROW || g.nodes[id].opcode == FS_REDUCE_COL; };
  // reductions by their direction in the work space (a row reduction of a flipped tensor runs down the columns)
  auto reduces_rows = [&](int id) { return is_reduce(id) && gp.kind[id] == KIND_COLV && C > 1; };   // lanes exchange values
  auto reduces_cols = [&](int id) { return is_reduce(id) && gp.kind[id] == KIND_ROWV && R > 1; };   // finished by the grid fold

  for (int m : gp.members) {
    const fs_node& n = g.nodes[m];
    const bool t = tf[m], t_op = n.opcode == FS_TRANSPOSE ? !t : t;
    const Kind result_kind = a.classify(n, t);
    if (n.opcode == FS_CONCAT) {
      // read from memory as one row out of two tensors; nothing is computed, so nothing is fused INTO a concat:
      // an operand produced by this group would have to exist in memory first
      if (t || result_kind != KIND_FULL) FS_FAIL(FS_ERR_UNSUPPORTED, "node %d (concat) does not fit the group's work space [%d,%d]", m, R, C);
      for (int k = 0; k < 2; ++k) {
        const int o = n.in[k];
        if (a.in_set[g.root_of[o]]) FS_FAIL(FS_ERR_UNSUPPORTED, "node %d (concat): operand %d is computed by the same kernel", m, o);
        for (const ExtTensor& e : gp.ext_in)
          if (e.node == o && e.kind != KIND_PART) FS_FAIL(FS_ERR_UNSUPPORTED, "node %d is read both whole and as part of a concat", o);
        add_ext_in(gp, o, KIND_PART, g.nodes[o].dtype);
        gp.kind[o] = KIND_PART;
      }
      gp.kind[m] = KIND_FULL;
      gp.level[m] = 0;
    }
    Kind operand_kind = result_kind;
    if (is_reduce(m) || n.opcode == FS_TRANSPOSE) operand_kind = KIND_FULL;
    if (result_kind == KIND_NONE || (n.opcode == FS_TRANSPOSE && result_kind != KIND_FULL))
      FS_FAIL(FS_ERR_UNSUPPORTED, "node %d [%d,%d] does not fit the group's work space [%d,%d]", m, n.rows, n.cols, R, C);
    gp.kind[m] = result_kind;
    const bool deferred = reduces_cols(m);
    int lvl = result_kind == KIND_ROWV && !deferred ? -1 : 0;
    for (int k = 0; k < n.num_in && n.opcode != FS_CONCAT; ++k) {
      Resolved r;
      if (g.flat_in[m][k]) {
        // a tensor in memory under another [rows, cols] label: the same elements at row * C + column of this work space.
        // It cannot come from this kernel's registers (another label means another assignment of elements to lanes).
        const int o = n.in[k];
        if (g.nodes[o].opcode == FS_CONST) continue;
        if (a.in_set[o] || a.in_set[g.root_of[o]])
          FS_FAIL(FS_ERR_UNSUPPORTED, "node %d reads node %d under another shape: it has to exist in memory first", m, o);
        if (t_op || operand_kind != KIND_FULL || (int64_t)g.nodes[o].rows * g.nodes[o].cols != (int64_t)R * C)
          FS_FAIL(FS_ERR_UNSUPPORTED, "node %d: operand %d (read as a flat element sequence) does not fill the work space [%d,%d]", m, o, R, C);
        for (const ExtTensor& e : gp.ext_in)
          if (e.node == o && e.kind != KIND_FULL) FS_FAIL(FS_ERR_UNSUPPORTED, "node %d is read in two ways", o);
        add_ext_in(gp, o, KIND_FULL, g.nodes[o].dtype);
        gp.kind[o] = KIND_FULL;
        continue;
      }
      if (!a.resolve(n.in[k], operand_kind, t_op, &r))
        FS_FAIL(FS_ERR_UNSUPPORTED, "node %d: operand %d does not fit the group's work space [%d,%d]", m, n.in[k], R, C);
      if (r.literal) continue;
      if (a.in_set[r.node]) {
        if (tf[r.node] != t_op) FS_FAIL(FS_ERR_UNSUPPORTED, "node %d mixes orientations", m);
        if (reduces_cols(r.node))
          FS_FAIL(FS_ERR_UNSUPPORTED, "node %d consumes node %d, whose value only exists after the whole grid has run", m, r.node);
        lvl = std::max(lvl, gp.level[r.node] + (reduces_rows(r.node) ? 1 : 0));
      } else {
        // a view of a value this kernel computes would have to exist in memory first
        if (a.in_set[g.root_of[r.node]]) FS_FAIL(FS_ERR_UNSUPPORTED, "node %d reads node %d, a view of a value computed by the same kernel", m, r.node);
        // tensors from memory: a full tensor can only be read in the orientation it is stored in
        if (r.kind == KIND_FULL && t_op) FS_FAIL(FS_ERR_UNSUPPORTED, "node %d would need a transposing load of node %d", m, r.node);
        for (const ExtTensor& e : gp.ext_in)
          if (e.node == r.node && e.kind != r.kind) FS_FAIL(FS_ERR_UNSUPPORTED, "node %d is read in two orientations", r.node);
        add_ext_in(gp, r.node, r.kind, g.nodes[r.node].dtype);
        gp.kind[r.node] = r.kind;
      }
    }
    gp.level[m] = lvl;
    if (reduces_rows(m)) gp.row_reduces.push_back(m);
    if (reduces_cols(m)) gp.col_reduces.push_back(m);

    // does the value leave the kernel?
    bool leaves = g.output_index[m] >= 0;
    std::function<void(int)> scan_users = [&](int id) {
      for (int u : g.users[id]) {
        const int uop = g.nodes[u].opcode;
        if (uop == FS_BCAST_ROWVEC || uop == FS_BCAST_COLVEC) scan_users(u);
        else if (op_is_view(uop)) leaves = true;  // a view is read from memory (or is a plan output): the value must exist there
        else if (!opt.clones) leaves |= !a.in_set[u];
        else {
          // every kernel that computes u reads m from memory unless it computes m itself
          const CloneInfo& ci = *opt.clones;
          auto needs = [&](int h) { return h == self_group ? !a.in_set[u] : (h >= 0 && !ci.computed_in(m, h)); };
          leaves |= needs(ci.group_of[u]);
          auto it = ci.extra.find(u);
          if (it != ci.extra.end())
            for (int h : it->second) leaves |= needs(h);
        }
      }
    };
    scan_users(m);
    // (a copy: the first kernel that computes the value is the one that stores it)
    if (opt.clones && opt.clones->group_of[m] != self_group) leaves = false;
    if (leaves) {
      ExtTensor e;
      e.node = m;
      e.kind = result_kind;
      e.dtype = n.dtype;
      e.transposed = t && result_kind == KIND_FULL && R > 1 && C > 1;
      e.deferred = deferred;
      if (t && result_kind == KIND_FULL && !e.transposed && (R > 1 || C > 1)) {
        // a flipped vector-shaped work space ([R,1] <-> [1,R]) has the same memory layout: plain store
      }
      gp.ext_out.push_back(e);
    }
  }
  if (gp.ext_out.empty()) FS_FAIL(FS_ERR_UNSUPPORTED, "group produces nothing");
  if ((int)(gp.ext_in.size() + gp.ext_out.size()) > kMaxGroupTensors) FS_FAIL(FS_ERR_UNSUPPORTED, "group touches too many tensors");

  // row reductions of one stage share one exchange
  std::map<int, int> per_level;
  for (int m : gp.row_reduces) gp.max_batched_reduces = std::max(gp.max_batched_reduces, ++per_level[gp.level[m]]);

  int arg = 0;
  for (ExtTensor& e : gp.ext_in) e.arg = arg++;
  for (ExtTensor& e : gp.ext_out) e.arg = arg++;
  // Tensors far larger than the caches are read / written once: keep them out of the way (non-temporal accesses).
  // So are smaller ones that no other kernel of the plan touches -- a plan input only this kernel reads, a plan output
  // nothing else in the plan consumes: what is written normally stays in the L2 until the end of the kernel and is
  // written back then, after the last wavefront, which costs a microsecond or two that a kernel of 5-10 us notices
  // (softmax f32 [4096,1024]: 8.0 -> 6.6 us, [2048,1024]: 5.8 -> 4.6 us; LayerNorm+GeLU bf16 [4096,1024]: 6.0 -> 5.1 us;
  // Adam [2048,2048]: 23.8 -> 21.2 us; 1 MB tensors: no difference).  Values that pass between kernels stay cacheable.
  constexpr uint64_t kStreamOnceBytes = 2ull << 20;
  auto bytes_of = [&](const ExtTensor& e) { return (uint64_t)g.nodes[e.node].rows * g.nodes[e.node].cols * dtype_size(e.dtype); };
  std::function<bool(int, bool)> used_only_here = [&](int id, bool live) {  // (live: nodes that no output needs do not count)
    for (int u : g.users[id]) {
      if (live && !g.live[u]) continue;
      const int uop = g.nodes[u].opcode;
      if (uop == FS_BCAST_ROWVEC || uop == FS_BCAST_COLVEC || op_is_view(uop)) {
        if (!used_only_here(u, live)) return false;  // (a view that is a plan output consumes nothing)
      } else if (!a.in_set[u]) {
        return false;
      }
    }
    return true;
  };
  for (ExtTensor& e : gp.ext_in) {
    const int root = g.root_of[e.node];
    const bool once = g.nodes[root].opcode == FS_INPUT && used_only_here(root, false);
    e.streaming = e.kind == KIND_FULL && bytes_of(e) >= (once ? kStreamOnceBytes : kStreamBytes);
  }
  for (ExtTensor& e : gp.ext_out) {
    const bool once = g.family_output[e.node] >= 0 && used_only_here(e.node, false);
    e.streaming = e.kind == KIND_FULL && !e.transposed && bytes_of(e) >= (once ? kStreamOnceBytes : kStreamBytes);
  }

  int min_es = 4;
  for (const ExtTensor& e : gp.ext_in)
    if (e.kind == KIND_FULL) min_es = std::min(min_es, dtype_size(e.dtype));
  gp.min_hbm_bytes = 0;
  for (const ExtTensor& e : gp.ext_in) gp.min_hbm_bytes += (uint64_t)g.nodes[e.node].rows * g.nodes[e.node].cols * dtype_size(e.dtype);
  for (const ExtTensor& e : gp.ext_out) gp.min_hbm_bytes += (uint64_t)g.nodes[e.node].rows * g.nodes[e.node].cols * dtype_size(e.dtype);
  // (an [R,C] value that another kernel reads is as a rule computed again there in the end: no reason to fold beside row reductions;
  // column sums and row norms f32 [3440,1000]: 17.5 us with one of two folds in the kernel of the norms, 11.4 apart in one launch)
  gp.fold_bytes = gp.min_hbm_bytes;
  for (const ExtTensor& e : gp.ext_out)
    if (e.kind == KIND_FULL && g.family_output[e.node] < 0) gp.fold_bytes -= bytes_of(e);
  gp.exchanges = false;
  gp.reads_alone = true;
  for (const ExtTensor& e : gp.ext_in) {
    const int root = g.root_of[e.node];
    gp.exchanges |= g.nodes[root].opcode != FS_INPUT;
    gp.reads_alone &= e.kind != KIND_FULL || (g.nodes[root].opcode == FS_INPUT && used_only_here(root, false));
  }
  for (const ExtTensor& e : gp.ext_out) gp.exchanges |= !used_only_here(e.node, true);

  // Elementwise groups whose tensors all are [R,C] need no rows: where those are no whole cache lines, the elements are cut into pieces of
  // kFlatPiece instead, whose accesses cover whole lines and whose lanes all have work; the last piece begins earlier and stores what it
  // shares with the one before it again.  dropout+residual fp32 [6115,2521] 38.7 -> 30.7 us, [26220,279] 18.3 -> 16.0, [4096,3000] 29.8 -> 24.8, bf16 [16384,4095] 87.3 -> 74.1,
  // [41282,43] 4.8 -> 3.8.  Not where rows are whole lines (as one row fp32 [5922,1088] 13.9 against 14.7, [65536,576] 74.3 and 75.5) or below 8 MB (no
  // difference).  Once the groups are final, and not where other kernels of the plan may take the same rows.
  bool flat = opt.grouped && (!opt.has_hint || opt.keep_flat) && !gp.exchanges && R > 1 && C > 1 && (int64_t)R * C < (1 << 30) && gp.min_hbm_bytes >= (8u << 20) && gp.row_reduces.empty() && gp.col_reduces.empty();
  int max_es = 1;
  for (int m : gp.members) flat &= gp.kind.at(m) == KIND_FULL && !tf[m] && g.nodes[m].opcode != FS_CONCAT;
  for (const auto* list : {&gp.ext_in, &gp.ext_out})
    for (const ExtTensor& e : *list) flat &= e.kind == KIND_FULL && !e.transposed, max_es = std::max(max_es, dtype_size(e.dtype));
  if (flat && (int64_t)C * max_es % 128 != 0) gp.flat = R * C;
  const fs_status st = choose_schedule(g, opt, &gp);
  // Rows that are no multiple of a vector long share cache lines with their neighbours, which other wavefronts read: ordinary
  // loads there.  LayerNorm+GeLU bf16 [30001,1021]: 24.5 -> 22.1 us right after the kernel that wrote the input (28.3 -> 28.7 us
  // from cold memory); masked softmax bf16 [32768,577] 22.5 -> 20.4 us (22.5 -> 22.8 us).  Not for groups that only stream
  // (no difference) or fold columns ([60001,515]: 33.3 -> 35.5 us).
  // Nor where a row has one such line among 32 or more and the tensors are far beyond the caches (masked softmax f32 [4096,8191]
  // 73.0 -> 68.2 us, softmax [9000,7001] 88.7 -> 83.6, residual+LayerNorm [3000,10001] 92.0 -> 90.4; but at 100 MB LayerNorm+GeLU
  // [4000,6001] 25.8 -> 27.4).  The narrow tiles of small column folds read with ordinary loads too.
  const bool long_rows = (int64_t)C * min_es >= 4096 && gp.min_hbm_bytes >= (128ull << 20);
  if (st == FS_OK && ((gp.s.shares_lines && !gp.row_reduces.empty() && gp.col_reduces.empty() && !long_rows) || (gp.s.narrow_tiles && gp.s.L < 32)))
    for (ExtTensor& e : gp.ext_in) e.streaming = false;
  if (st == FS_OK && gp.s.chunked)  // every stage reads the row again: keep it in the caches
    for (ExtTensor& e : gp.ext_in) e.streaming = false;
  return st;
}

// -------------------------------------------------------------------------------------------
// Schedule tuning (Section 4.3): candidates and the library-driven choice.
// -------------------------------------------------------------------------------------------
std::vector<fs_sched_hint> candidate_hints(const GroupPlan& base) {
  const Schedule& s = base.s;
  std::vector<fs_sched_hint> out;
  if (s.chunked) return out;  // one row per 1024-lane workgroup: nothing to vary
  std::vector<int> Ls, WGs, caps;
  for (int L : {s.L / 2, s.L, s.L * 2})
    if (L >= 1 && L <= 1024) Ls.push_back(L);
  for (int WG : {s.WG / 2, s.WG, s.WG * 2})
    if (WG >= 64 && WG <= 1024) WGs.push_back(WG);
  caps.push_back(0);
  if (!base.col_reduces.empty() && s.grid > 1)  // every workgroup leaves a partial: the grid is a real trade-off
    for (int c : {s.grid / 2, s.grid * 2})
      if (c >= 1 && c <= 2048) caps.push_back(c);
  for (int L : Ls)
    for (int WG : WGs)
      for (int cap : caps) {
        if (WG < L) continue;
        if (L == s.L && WG == s.WG && cap == 0) continue;  // the base schedule itself
        out.push_back(fs_sched_hint{L, WG, cap, 0});
      }
  // narrow column tiles: the other numbers of trips in flight
  for (int u : {1, 2, 4})
    if (s.narrow_tiles && u != s.U) out.push_back(fs_sched_hint{s.L, s.WG, 0, u});
  // looping kernels: the other number of row tiles per trip with the base shape
  if (!s.narrow_tiles && s.grid < s.n_iters && s.CT == 1) out.push_back(fs_sched_hint{s.L, s.WG, 0, s.U == 1 ? 2 : 1});
  // row-reduction groups with [1,C] operands staged in LDS: one trip per workgroup against looping
  // workgroups that stage once (32 wavefronts per CU), whichever the base is not
  if (s.stage_rowv && base.col_reduces.empty() && s.CT == 1 && s.L <= 256) {
    const int wg_loop = s.L >= 128 ? std::min(1024, 4 * s.L) : 1024, wg_once = std::max(256, 4 * s.L);
    if (s.grid >= s.n_iters) out.push_back(fs_sched_hint{s.L, wg_loop, (int)(device_limits().resident_lanes / wg_loop), 0});
    else if (wg_once <= 1024) out.push_back(fs_sched_hint{s.L, wg_once, 1 << 20, 0});
  }
  return out;
}

bool choose_from_library(const Graph& g, const std::vector<int>& members, const std::vector<int>& group_of, int self_group,
                         const PlanOptions& opt, GroupPlan* gp) {
  // a candidate has to beat the analytic schedule by more than the noise of the measurement
  constexpr double kMargin = 0.95;
  double best = 0.0;
  const bool base_known = perflib_lookup(perf_key(*gp), &best);
  best *= kMargin;
  bool changed = false;
  GroupPlan cand;
  const std::vector<fs_sched_hint> hints = candidate_hints(*gp);
  for (const fs_sched_hint& h : hints) {
    PlanOptions o = opt;
    o.hint = h;
    o.has_hint = true;
    if (analyse_group(g, members, group_of, self_group, o, &cand) != FS_OK) continue;
    if (cand.s.L != h.lanes_per_row || cand.s.WG != h.wg_threads) continue;  // the hint was not legal for this group
    if (generate_kernel(g, &cand, self_group) != FS_OK) continue;
    double us = 0.0;
    if (!perflib_lookup(perf_key(cand), &us)) continue;
    // an unmeasured base schedule is not displaced: only compare within the library
    if (!base_known) continue;
    if (us < best) {
      best = us;
      *gp = cand;
      changed = true;
    }
  }
  return changed;
}

// -------------------------------------------------------------------------------------------
// Group formation.
//
// Unfused mode: one group per compute node.  Caller-given plan: checked, not changed.
// Otherwise a greedy producer/consumer fusion in the spirit of Algorithm 1 (Section 3.2):
// nodes are visited from the outputs upwards (the order of decreasing span); a node joins the
// group of one of its users when the three conditions of SchdConsistent hold:
//   1. no dependence cycle between groups would appear (the paper's `giveup` test),
//   2. it has a user in that group (producer/consumer fusion only),
//   3. the merged group still has a valid schedule and fits the LDS budget (analyse_group).
// -------------------------------------------------------------------------------------------
namespace {

// Performance feedback to the fusion decision (the role of the schedule planner's feedback edge,
// Section 2.2): a column reduction finished inside a kernel costs a ticketed grid-wide fold, a few
// microseconds of latency.  That is hidden behind the streaming of a large group, but for a
// launch-bound group it is dearer than the launch it saves, so small groups do not take one in.
bool worth_fusing(const GroupPlan& merged, bool apart) {
  constexpr uint64_t kFoldWorthBytes = 16ull << 20;
  // A transposed root that cannot leave through an LDS tile (rows spread over a whole workgroup)
  // is written element by element, R elements apart: an order of magnitude slower than handing
  // the value to a kernel of its own that transposes in 2-D tiles (softmax + transpose of
  // [8192,4096]: 408 us fused, 95 us as two kernels); launch-bound groups keep it (one launch less).
  if (merged.members.size() > 1 && !merged.s.tile_transpose && !merged.s.tiled_transpose && merged.min_hbm_bytes >= kFoldWorthBytes)
    for (const ExtTensor& e : merged.ext_out)
      if (e.transposed) return false;
  // A handful of very long rows: one workgroup per row leaves most of the device idle, so such a
  // group, if its rows do not fit one workgroup's registers either, is only formed when its rows can
  // be split over workgroups.  Softmax of [8, 1M]: 286 us as
  // one kernel on 8 CUs, 38 us as three kernels that each fill the device; [32, 256K]: 73 -> 37 us;
  // from 64 rows on the single kernel is as fast or faster ([128, 64K]: 20 against 35 us).
  if (merged.members.size() > 1 && merged.s.few_long_rows && !merged.s.split_rows && merged.s.chunked && merged.R <= 32) return false;
  // Narrow column tiles fold little, or side by side; what feeds their reductions, and further reductions of the same tensors,
  // join them at any size (column sums, maxima and row norms f32 [421,192] in three kernels 16.1 us, in two 7.2; [20000,64], whose
  // tiles fold in two levels, 18.5 and 10.7).  Not where the reductions are row reductions of transposed tensors: there the other consumers want
  // the rows in one workgroup (the 200-node DAG: 29.4 us with those kept apart, 30.6 us without).
  bool narrow = merged.s.narrow_tiles;
  for (const auto& f : merged.tflag) narrow &= !f.second;
  // A group that stores several values transposed and exchanges values with others gives up its place in a chain of groups for a fold, and has
  // few workgroups left for those values: from 64 MB on.  Random DAG of 200 ops [2000,256] 44.2 -> 33.3 us, [2048,256] 41.5 -> 30.1, [2048,384] 50.3 -> 39.6.
  int flipped = 0;
  for (const ExtTensor& e : merged.ext_out) flipped += e.transposed;
  // Beside row reductions the fold costs what a workgroup's partial weighs, which is what a row holds, and a kernel of its own costs another
  // read of the rows.  Tall tensors pay from 8.5 MB on (column sums + row norms fp32 [65536,33] 14.4 us in kernels side by side, 10.0 in one,
  // [16384,200] 12.4 and 10.3, LayerNorm backward [16384,64] 12.9 and 9.5; [16384,128], 8.4 MB, 8.0 and 8.7; [8192,300] 9.2 and 10.5), unless values leave
  // transposed (row softmax numerators, transposed, with their column sums [9000,150] 9.0 apart and 12.4 in one, [11403,64] 7.1 and 9.3).  Below 2048 rows the fold weighs
  // more than the read, to 32 MB, as long as the kernels only read the same tensors (apart, folds_exchange_rows: [1421,3392] 13.3 and 16.0, [1000,5000] 11.4
  // and 17.3, LayerNorm backward [400,5000] 12.3 and 17.3, [1300,2000] 15.3 and 18.3, [300,8192] 12.8 and 18.6; but [1500,8000], 48 MB, 30.8 and 23.2, LayerNorm
  // backward [1500,3000], 54 MB, 25.2 and 20.4).
  const uint64_t beside = merged.R >= 8192 && flipped == 0 ? 8500000 : merged.R >= 2048 || !apart ? kFoldWorthBytes : 32000000;
  const uint64_t worth = flipped >= 2 && merged.exchanges && !merged.row_reduces.empty() ? 64ull << 20 : merged.row_reduces.empty() ? kFoldWorthBytes : beside;
  return merged.col_reduces.empty() || merged.members.size() == 1 || merged.s.grid == 1 || narrow || (merged.row_reduces.empty() ? merged.min_hbm_bytes : merged.fold_bytes) >= worth;
}

struct Former {
  const Graph& g;
  const PlanOptions& opt;
  std::vector<int> group_of;              // node -> group id, -1 unassigned/free
  std::vector<std::vector<int>> members;  // group id -> nodes
  std::vector<char> live;

  Former(const Graph& g_, const PlanOptions& o) : g(g_), opt(o), group_of(g_.n(), -1), live(g_.n(), 0) {}

  void mark_live() {
    std::vector<int> stack(g.outputs.begin(), g.outputs.end());
    while (!stack.empty()) {
      const int id = stack.back();
      stack.pop_back();
      if (live[id]) continue;
      live[id] = 1;
      for (int k = 0; k < g.nodes[id].num_in; ++k) stack.push_back(g.nodes[id].in[k]);
    }
  }

  // compute-node users of `id`, looking through broadcasts
  void real_users(int id, std::vector<int>* out) const {
    for (int u : g.users[id]) {
      if (!live[u]) continue;
      const int uop = g.nodes[u].opcode;
      if (uop == FS_BCAST_ROWVEC || uop == FS_BCAST_COLVEC || op_is_view(uop)) real_users(u, out);
      else out->push_back(u);
    }
  }

  // is group `to` reachable from group `from` along producer -> consumer edges?
  bool reaches(int from, int to) const {
    std::vector<char> seen(members.size(), 0);
    std::vector<int> stack{from};
    while (!stack.empty()) {
      const int grp = stack.back();
      stack.pop_back();
      if (grp == to) return true;
      if (seen[grp]) continue;
      seen[grp] = 1;
      for (int m : members[grp]) {
        std::vector<int> us;
        real_users(m, &us);
        for (int u : us)
          if (group_of[u] >= 0 && group_of[u] != grp && !seen[group_of[u]]) stack.push_back(group_of[u]);
      }
    }
    return false;
  }

  // direct producer -> consumer successors of a group
  std::set<int> successors(int grp) const {
    std::set<int> out;
    for (int m : members[grp]) {
      std::vector<int> us;
      real_users(m, &us);
      for (int u : us)
        if (group_of[u] >= 0 && group_of[u] != grp) out.insert(group_of[u]);
    }
    return out;
  }

  // Second pass: fuse groups that are not (only) producer and consumer of each other.  This is
  // the role of the paper's intra-layer ElementwiseFusion and of its multi-root computations
  // (Sections 3.2 and 4.3): kernels over the same work space are merged when they read a common
  // [R,C] tensor (one read instead of two) or when they are so small that the launch, not the
  // traffic, is what they cost (the tunable footprint threshold of Section 3.2).
  void merge_siblings() {
    constexpr uint64_t kFootprintThreshold = 16ull << 20;
    std::vector<GroupPlan> plan(members.size());
    std::vector<char> valid(members.size(), 0);
    auto analyse = [&](int grp) {
      valid[grp] = !members[grp].empty() && analyse_group(g, members[grp], group_of, grp, opt, &plan[grp]) == FS_OK;
    };
    for (size_t grp = 0; grp < members.size(); ++grp) analyse((int)grp);
    // The scan restarts from the first pair after every merge (which merge comes first decides the result: merging
    // is not confluent), but a pair whose merged group was analysed and refused is not analysed again until one of
    // the two groups has changed: the analysis is the expensive part, and it depends on the two member sets only.
    std::vector<int> version(members.size(), 0);
    std::map<std::pair<size_t, size_t>, std::pair<int, int>> refused;
    bool changed = true;
    GroupPlan merged_plan;
    while (changed) {
      changed = false;
      for (size_t a = 0; a < members.size() && !changed; ++a) {
        if (!valid[a]) continue;
        for (size_t b = a + 1; b < members.size() && !changed; ++b) {
          if (!valid[b]) continue;
          // work spaces must nest: equal, or one of them is a vector ([R,1] / [1,C]) of the other
          auto fits = [](int x, int y) { return x == y || x == 1 || y == 1; };
          // ... or do so after a flip (a transpose inside the merged group reorients one side)
          const bool straight = fits(plan[a].R, plan[b].R) && fits(plan[a].C, plan[b].C);
          const bool flipped = fits(plan[a].R, plan[b].C) && fits(plan[a].C, plan[b].R);
          if (!straight && !flipped) continue;
          if ((int)(members[a].size() + members[b].size()) > kMaxGroupMembers) continue;
          // profitable?
          bool share_full = false;
          for (const ExtTensor& x : plan[a].ext_in)
            for (const ExtTensor& y : plan[b].ext_in) share_full |= x.node == y.node && x.kind == KIND_FULL && y.kind == KIND_FULL;
          for (const ExtTensor& x : plan[a].ext_out)
            for (const ExtTensor& y : plan[b].ext_in) share_full |= x.node == y.node && y.kind == KIND_FULL;
          for (const ExtTensor& x : plan[b].ext_out)
            for (const ExtTensor& y : plan[a].ext_in) share_full |= x.node == y.node && y.kind == KIND_FULL;
          const bool small = plan[a].min_hbm_bytes + plan[b].min_hbm_bytes <= kFootprintThreshold;
          if (!share_full && !small) continue;
          auto seen = refused.find({a, b});
          if (seen != refused.end() && seen->second == std::make_pair(version[a], version[b])) continue;
          // a path a -> c -> ... -> b through a third group would become a cycle
          bool cycle = false;
          for (int c : successors((int)a)) cycle |= c != (int)b && reaches(c, (int)b);
          for (int c : successors((int)b)) cycle |= c != (int)a && reaches(c, (int)a);
          if (cycle) continue;
          std::vector<int> merged = members[a];
          merged.insert(merged.end(), members[b].begin(), members[b].end());
          if (analyse_group(g, merged, group_of, (int)a, opt, &merged_plan) != FS_OK || !worth_fusing(merged_plan, opt.folds_apart)) {
            refused[{a, b}] = {version[a], version[b]};
            continue;
          }
          ++version[a];
          for (int m : members[b]) group_of[m] = (int)a;
          members[a] = merged;
          members[b].clear();
          valid[b] = 0;
          plan[a] = merged_plan;
          changed = true;
        }
      }
    }
  }

  // ---- Work/Span analysis (Section 3.1) --------------------------------------------------------
  // span = 0 for a node nothing live consumes (a root); otherwise 1 + the largest span among its
  // users (broadcasts are looked through: they are inlined, not instructions of their own).
  // Nodes of equal span form a layer and do not depend on each other.
  std::vector<int> spans() const {
    std::vector<int> span(g.n(), -1);
    for (int id = g.n() - 1; id >= 0; --id) {
      if (!live[id] || op_is_free(g.nodes[id].opcode)) continue;
      std::vector<int> us;
      real_users(id, &us);
      int sp = 0;
      for (int u : us) sp = std::max(sp, span[u] + 1);
      span[id] = sp;
    }
    return span;
  }

  static bool is_elementwise(int op) { return op_is_unary(op) || op_is_binary(op) || op == FS_CMP || op == FS_SELECT; }

  // ---- the layered planner: Section 3.2 as written ----------------------------------------------
  // For every layer from the roots upwards: (1) intra-layer ElementwiseFusion of the layer's still
  // unassigned elementwise nodes (schedule-compatible, fused footprint under the threshold);
  // (2) for every fusion root of the layer, Algorithm 1: walk the layers above it, fuse a node
  // when SchdConsistent holds, otherwise put it in `giveup`.
  void plan_layered() {
    constexpr uint64_t kFootprintThreshold = 16ull << 20;
    const std::vector<int> span = spans();
    int max_span = -1;
    for (int sp : span) max_span = std::max(max_span, sp);
    std::vector<std::vector<int>> layer(max_span + 1);
    for (int id = 0; id < g.n(); ++id)
      if (span[id] >= 0) layer[span[id]].push_back(id);
    GroupPlan scratch;
    for (int s = 0; s <= max_span; ++s) {
      // (1) ElementwiseFusion among the unassigned nodes of this layer
      std::vector<int> roots;  // group ids created in this layer
      for (int id : layer[s]) {
        if (group_of[id] >= 0) continue;
        int joined = -1;
        if (is_elementwise(g.nodes[id].opcode)) {
          for (int grp : roots) {
            if (!is_elementwise(g.nodes[members[grp][0]].opcode)) continue;
            std::vector<int> merged = members[grp];
            merged.push_back(id);
            if (analyse_group(g, merged, group_of, grp, opt, &scratch) != FS_OK) continue;
            if (scratch.min_hbm_bytes > kFootprintThreshold) continue;
            joined = grp;
            break;
          }
        }
        if (joined < 0) {
          joined = (int)members.size();
          members.push_back({});
          roots.push_back(joined);
        }
        group_of[id] = joined;
        members[joined].push_back(id);
      }
      // (2) Algorithm 1 from every fusion root of this layer
      for (int grp : roots) {
        std::set<int> giveup;
        for (int l = s + 1; l <= max_span; ++l) {
          for (int hlo : layer[l]) {
            if (group_of[hlo] >= 0) continue;
            std::vector<int> us;
            real_users(hlo, &us);
            bool user_gave_up = false, user_fused = false;
            for (int u : us) {
              user_gave_up |= giveup.count(u) != 0;
              user_fused |= group_of[u] == grp;
            }
            bool ok = !user_gave_up && user_fused;  // SchdConsistent, tests 1 and 2
            if (ok) {
              // (exact form of test 1 for users that already belong to other fused computations)
              for (int u : us) {
                const int h = group_of[u];
                if (h >= 0 && h != grp && reaches(h, grp)) ok = false;
              }
            }
            if (ok) {  // test 3: an optimised schedule (and LDS plan) for the fused computation exists
              std::vector<int> merged = members[grp];
              merged.push_back(hlo);
              ok = (int)merged.size() <= 96 && analyse_group(g, merged, group_of, grp, opt, &scratch) == FS_OK && worth_fusing(scratch, opt.folds_apart);
            }
            if (ok) {
              group_of[hlo] = grp;
              members[grp].push_back(hlo);
            } else {
              giveup.insert(hlo);
            }
          }
        }
      }
    }
  }

  fs_status topo_order(std::vector<std::vector<int>>* ordered) const {
    const int NG = (int)members.size();
    std::vector<std::set<int>> succ(NG);
    std::vector<int> indeg(NG, 0);
    for (int grp = 0; grp < NG; ++grp)
      for (int m : members[grp]) {
        std::vector<int> us;
        real_users(m, &us);
        for (int u : us) {
          const int h = group_of[u];
          if (h >= 0 && h != grp && succ[grp].insert(h).second) ++indeg[h];
        }
      }
    // Kahn, smallest first-member id first (stable, close to the caller's order)
    auto key = [&](int grp) { return *std::min_element(members[grp].begin(), members[grp].end()); };
    std::set<std::pair<int, int>> ready;
    for (int grp = 0; grp < NG; ++grp)
      if (!members[grp].empty() && indeg[grp] == 0) ready.insert({key(grp), grp});
    size_t placed = 0, nonempty = 0;
    for (int grp = 0; grp < NG; ++grp) nonempty += !members[grp].empty();
    while (!ready.empty()) {
      const int grp = ready.begin()->second;
      ready.erase(ready.begin());
      ordered->push_back(members[grp]);
      ++placed;
      for (int h : succ[grp])
        if (--indeg[h] == 0) ready.insert({key(h), h});
    }
    if (placed != nonempty) FS_FAIL(FS_ERR_UNSUPPORTED, "the grouping has a dependence cycle between groups");
    return FS_OK;
  }
};

}  // namespace

fs_status form_groups(const Graph& g, const fs_graph_desc* desc, const PlanOptions& opt, std::vector<int>* group_of,
                      std::vector<std::vector<int>>* ordered) {
  Former f(g, opt);
  f.mark_live();
  const int N = g.n();
  GroupPlan scratch;

  if (opt.mode == FS_MODE_UNFUSED) {
    for (int id = 0; id < N; ++id)
      if (f.live[id] && !op_is_free(g.nodes[id].opcode)) {
        f.group_of[id] = (int)f.members.size();
        f.members.push_back({id});
      }
  } else if (desc->group_of_node) {
    std::map<int, int> remap;
    for (int id = 0; id < N; ++id) {
      if (!f.live[id] || op_is_free(g.nodes[id].opcode)) continue;
      const int want = desc->group_of_node[id];
      if (want < 0) FS_FAIL(FS_ERR_INVALID_ARG, "group_of_node[%d] = %d", id, want);
      auto it = remap.find(want);
      if (it == remap.end()) {
        it = remap.insert({want, (int)f.members.size()}).first;
        f.members.push_back({});
      }
      f.group_of[id] = it->second;
      f.members[it->second].push_back(id);
    }
  } else if (opt.layered) {
    f.plan_layered();
  } else {
    for (int id = N - 1; id >= 0; --id) {
      if (!f.live[id] || op_is_free(g.nodes[id].opcode)) continue;
      std::vector<int> us;
      f.real_users(id, &us);
      // candidate groups: those of its users, most users first
      std::map<int, int> votes;
      for (int u : us)
        if (f.group_of[u] >= 0) ++votes[f.group_of[u]];
      std::vector<std::pair<int, int>> cands;
      for (auto& kv : votes) cands.push_back({-kv.second, kv.first});
      std::sort(cands.begin(), cands.end());
      int joined = -1;
      for (auto& cand : cands) {
        const int grp = cand.second;
        // condition 1: joining must not close a cycle through a user left outside
        bool cycle = false;
        for (int u : us) {
          const int h = f.group_of[u];
          if (h >= 0 && h != grp && f.reaches(h, grp)) {
            cycle = true;
            break;
          }
        }
        if (cycle) continue;
        // condition 3: schedule and LDS plan of the merged group
        std::vector<int> merged = f.members[grp];
        merged.push_back(id);
        if ((int)merged.size() > kMaxGroupMembers) continue;
        if (analyse_group(g, merged, f.group_of, grp, opt, &scratch) != FS_OK) continue;
        if (!worth_fusing(scratch, opt.folds_apart)) continue;
        joined = grp;
        break;
      }
      if (joined < 0) {
        joined = (int)f.members.size();
        f.members.push_back({});
      }
      f.group_of[id] = joined;
      f.members[joined].push_back(id);
    }
    f.merge_siblings();
  }
  *group_of = f.group_of;
  return f.topo_order(ordered);
}

void recompute_across_kernels(const Graph& g, const PlanOptions& opt, std::vector<int>* group_of,
                              std::vector<std::vector<int>>* ordered, CloneInfo* ci) {
  const int NG = (int)ordered->size();
  ci->group_of = *group_of;
  ci->extra.clear();
  if (NG < 2) return;
  PlanOptions o = opt;
  o.clones = ci;
  std::vector<GroupPlan> gps(NG);
  for (int gi = 0; gi < NG; ++gi)
    if (analyse_group(g, (*ordered)[gi], *group_of, gi, o, &gps[gi]) != FS_OK) return;  // (plan creation reports it)
  auto elementwise = [&](int op) { return op_is_unary(op) || op_is_binary(op) || op == FS_CMP || op == FS_SELECT; };
  auto in_list = [](const std::vector<ExtTensor>& l, int node) {
    for (const ExtTensor& e : l)
      if (e.node == node) return true;
    return false;
  };
  for (int b = 1; b < NG; ++b) {
    for (int round = 0; round < 16; ++round) {  // a copy may expose its own producer
      bool changed = false;
      const std::vector<ExtTensor> reads = gps[b].ext_in;
      for (const ExtTensor& e : reads) {
        const int t = e.node;
        const fs_node& n = g.nodes[t];
        if (e.kind != KIND_FULL || ci->group_of[t] < 0 || !elementwise(n.opcode) || ci->computed_in(t, b)) continue;
        if (g.family_output[t] >= 0) continue;  // a plan output exists in memory anyway: reading it is as cheap as its operands
        // every reader inside b takes it as a plain operand (not under another shape), and nobody views it
        bool plain = true;
        for (int u : g.users[t]) plain &= !op_is_view(g.nodes[u].opcode);
        for (int m : (*ordered)[b])
          for (int k = 0; k < g.nodes[m].num_in; ++k) plain &= !(g.nodes[m].in[k] == t && g.flat_in[m][k]);
        if (!plain) continue;
        // the value and, with it, those of its elementwise producers that exist in no memory: everything else they read has to
        // be there already (plan inputs, values some kernel stores anyway, vectors)
        std::vector<int> T, stack{t};
        bool available = true;
        while (!stack.empty() && available) {
          const int x = stack.back();
          stack.pop_back();
          if (std::find(T.begin(), T.end(), x) != T.end()) continue;
          T.push_back(x);
          if (T.size() > 8) available = false;
          const fs_node& xn = g.nodes[x];
          for (int k = 0; k < xn.num_in && available; ++k) {
            int src = xn.in[k];
            if (g.flat_in[x][k]) available = false;
            while (g.nodes[src].opcode == FS_BCAST_ROWVEC || g.nodes[src].opcode == FS_BCAST_COLVEC) src = g.nodes[src].in[0];
            const fs_node& sn = g.nodes[src];
            if (sn.opcode == FS_CONST || sn.opcode == FS_INPUT) continue;
            const int h = ci->group_of[src];
            if (h >= 0 && ci->computed_in(src, b)) continue;
            if (h < 0 || h >= b) available = false;  // (a view; or not a value of an earlier kernel)
            else if (in_list(gps[h].ext_out, src)) continue;
            else if ((int64_t)sn.rows * sn.cols < (int64_t)n.rows * n.cols) continue;  // a vector: storing it costs next to nothing
            else if (elementwise(sn.opcode)) stack.push_back(src);
            else available = false;
          }
        }
        // (bytes are what is scarce, but not free of charge: at most two transcendental or division-like operations are
        // computed a second time for one value)
        int dear = 0;
        for (int x : T) dear += op_is_approx(g.nodes[x].opcode) || g.nodes[x].opcode == FS_DIV || g.nodes[x].opcode == FS_SQRT;
        if (!available || dear > 2) continue;
        // every producer keeps what it still uses itself
        CloneInfo trial = *ci;
        std::map<int, std::vector<int>> mm;  // member lists of the kernels that change
        mm[b] = (*ordered)[b];
        std::sort(T.begin(), T.end());
        for (int i = (int)T.size() - 1; i >= 0; --i) {  // consumers before producers
          const int x = T[i], a = trial.group_of[x];
          if (!mm.count(a)) mm[a] = (*ordered)[a];
          std::vector<int>& ma = mm[a];
          // it stays in its kernel while something there uses it, or while a third kernel reads it from memory
          // (the first kernel that computes a value is the one that stores it, and that one runs before every reader)
          bool stays = false;
          for (int u : g.users[x]) {
            std::vector<int> chain{u};
            while (!chain.empty()) {
              const int y = chain.back();
              chain.pop_back();
              const int yop = g.nodes[y].opcode;
              if (yop == FS_BCAST_ROWVEC || yop == FS_BCAST_COLVEC) {
                chain.insert(chain.end(), g.users[y].begin(), g.users[y].end());
                continue;
              }
              stays |= std::find(ma.begin(), ma.end(), y) != ma.end() || op_is_view(yop);
              auto other = [&](int h) { return h >= 0 && h != a && h != b && !trial.computed_in(x, h); };
              stays |= other(trial.group_of[y]);
              auto it = trial.extra.find(y);
              if (it != trial.extra.end())
                for (int h : it->second) stays |= other(h);
            }
          }
          mm[b].push_back(x);
          if (stays) {
            trial.extra[x].insert(b);
          } else {
            ma.erase(std::find(ma.begin(), ma.end(), x));
            trial.group_of[x] = b;
            trial.extra[x].erase(b);
          }
        }
        bool fits = (int)mm[b].size() <= kMaxGroupMembers;
        for (auto& kv : mm) fits &= !kv.second.empty();
        if (!fits) continue;
        PlanOptions ot = opt;
        ot.clones = &trial;
        std::map<int, GroupPlan> np;
        uint64_t before = 0, after = 0;
        for (auto& kv : mm) {
          fits = fits && analyse_group(g, kv.second, trial.group_of, kv.first, ot, &np[kv.first]) == FS_OK;
          if (!fits) break;
          before += gps[kv.first].min_hbm_bytes;
          after += np[kv.first].min_hbm_bytes;
        }
        if (!fits || after >= before || !worth_fusing(np[b], opt.folds_apart)) continue;
        // a kernel that changes its form for the copy (rows no longer held in registers, another launch shape class) is not worth it
        if (np[b].s.chunked != gps[b].s.chunked || np[b].s.split_rows != gps[b].s.split_rows || np[b].s.col_tiled != gps[b].s.col_tiled) continue;
        for (auto& kv : mm) {
          (*ordered)[kv.first] = kv.second;
          gps[kv.first] = np[kv.first];
        }
        *ci = trial;
        changed = true;
        break;
      }
      if (!changed) break;
    }
  }
  *group_of = ci->group_of;
}

// -------------------------------------------------------------------------------------------
// Groups joined over their column reductions (GroupPlan::joined).
// -------------------------------------------------------------------------------------------
namespace {

// 32-bit registers of rows that a lane may hold, by the workgroup that a compute unit runs: of 256 at 512 lanes.  (Batch
// normalisation f32 compiles without scratch up to here; where another body does not, plan creation gives the joined kernel up.)
constexpr int kJoinRegs = 200;

// Lanes of a tile, workgroup, workgroups per tile, rows per lane.  Batch normalisation f32, us:
//  - 8 lanes, one 128-byte run of f32, where rows are whole cache lines ([16384,1024] 27.0, 27.2 of 16 lanes, 27.8 of 32;
//    [1000,8192] 12.5, 13.6 of 16) and in narrow rows ([30000,33] 12.3 of 8, 13.5 of 16; [5000,48] 7.2, 7.7); elsewhere tiles share
//    the lines at their edges: 16 lanes below 8 MB ([3000,200] 8.5 of 8, 8.4 of 16; [1000,1000] 7.5, 7.2, 7.7 of 32), 32 above ([8000,2000] 32.1 of
//    8, 28.8 of 16; [2000,3001] 25.7, 19.8, 16.5 of 32; [25000,300] 31.5, 25.8, 24.4; [65536,99] 33.9, 29.3, 26.7).
//  - One workgroup to a tile of up to 96 KB, which then meets nobody: [600,600] 5.6 us of one, 6.9 of four; [333,777] 5.3, 7.1;
//    but 128 KB, [1000,1000], 9.6 of one, 7.4 of eight.  Tiles of half the width where that makes them small enough and the tensor
//    is below 2 MB ([1500,100] 5.5, 6.5 of 8 lanes; above, 64-byte runs cost more, [1000,1000] 7.9).
//  - Larger tiles: as many workgroups as fill the device, each with 16 KB or more of the tile ([8192,16] 7.2 us of 16, 7.6 of 32,
//    9.7 of 64), 32 at most, up to 128 where each would have more than 200 KB ([40000,128], 160 KB, 13.9 of 32, 14.0 of 64;
//    [65536,64], 256 KB, 16.0 and 13.9; [65536,99] on tiles of 32 lanes 26.7 of 128, 29.6 of 256): the counts of a tile queue up.
//  - 256 lanes, two workgroups to a compute unit, or 512, one, from 8 MB on, where half as many partials count ([2000,3001]
//    16.9 and 16.5; [16384,1024] 27.4 and 27.0; [4096,1024] 10.2 either way).
// Three kernels before: [16384,1024] 52, [2500,8192] 73, [4096,1024] 19.3, [65536,99] 29.9, [2000,3001] 27.2, [300,64] 10.1 (joined 4.7).
fs_status pick_join_shape(GroupPlan* gp, int dwords_per_row, int max_es) {
  Schedule& s = gp->s;
  const int R = gp->R, CUS = device_limits().cus;
  const int64_t run = (int64_t)s.V * max_es, row = (int64_t)gp->C * max_es, bytes = R * row;  // of the widest tensor: what a lane takes of a row, a row, all
  auto tile_bytes = [&](int lanes) { return R * std::min(lanes, pow2_ceil(s.NV)) * run; };
  int L = 8;
  const bool half = tile_bytes(8) > 96 << 10 && tile_bytes(4) <= 96 << 10 && bytes <= 2 << 20, alone = half || tile_bytes(8) <= 96 << 10;
  if (half) L = 4;
  else if (!alone && row % 128 != 0 && s.NV > 16) L = bytes >= 8 << 20 ? 32 : 16;
  L = std::min(L, pow2_ceil(s.NV));
  int WG = bytes >= 8 << 20 ? 512 : 256;
  WG = std::max(64, std::min(WG, L * pow2_ceil(std::min(R, 1024))));
  const int G = WG / L, CT = (s.NV + L - 1) / L, trips = (R + G - 1) / G;
  int RB = 1;
  if (!alone) {
    int most = 32;
    while (most < 128 && tile_bytes(L) / most > 200 << 10) most *= 2;
    RB = std::max(1, std::min({CUS * 512 / WG / CT, (int)std::min<int64_t>(tile_bytes(L) >> 14, 1024), most, trips}));
  }
  const int U = (trips + RB - 1) / RB;
  s.L = L, s.NVL = 1, s.E = s.V, s.WG = WG, s.G = G, s.CT = CT, s.n_iters = trips, s.RB = (trips + U - 1) / U, s.U = U;
  s.grid = CT * s.RB;
  s.fold_width = s.fold_piece = L * s.V;
  if (U * dwords_per_row > kJoinRegs) FS_FAIL(FS_ERR_UNSUPPORTED, "%d rows to a lane do not fit its registers", U);
  return FS_OK;
}

}  // namespace

fs_status join_groups(const Graph& g, const std::vector<GroupPlan>& groups, int first, int count, const PlanOptions& opt, GroupPlan* out) {
  GroupPlan& gp = *out;
  gp = GroupPlan();
  gp.joined = true;
  std::set<int> members;
  for (int k = first; k < first + count; ++k) {
    const GroupPlan& p = groups[k];
    members.insert(p.members.begin(), p.members.end());
    gp.R = std::max(gp.R, p.R), gp.C = std::max(gp.C, p.C);
    for (const auto& t : p.tflag)
      if (t.second) FS_FAIL(FS_ERR_UNSUPPORTED, "a transposed value");
  }
  gp.members.assign(members.begin(), members.end());
  if (gp.R < 2 || gp.C < 2 || (int)gp.members.size() > kMaxGroupMembers) FS_FAIL(FS_ERR_UNSUPPORTED, "nothing to join");
  Analyser a(g, gp);
  for (int m : gp.members) a.in_set[m] = 1;
  a.R = gp.R, a.C = gp.C;
  bool folds = false;
  for (int m : gp.members) folds |= g.nodes[m].opcode == FS_REDUCE_COL;
  if (!folds) FS_FAIL(FS_ERR_UNSUPPORTED, "no column reduction");
  auto read_by_others = [&](int id) {  // from memory, by groups that are not joined here
    for (int k = 0; k < (int)groups.size(); ++k)
      if (k < first || k >= first + count)
        for (const ExtTensor& e : groups[k].ext_in)
          if (g.root_of[e.node] == id) return true;
    return false;
  };
  int top = 0, max_es = 0, dwords = 0;
  for (int m : gp.members) {
    const fs_node& n = g.nodes[m];
    const bool reduce = n.opcode == FS_REDUCE_COL;
    const Kind k = a.classify(n.rows, n.cols);
    if ((k != KIND_FULL && k != KIND_ROWV) || n.opcode == FS_REDUCE_ROW || n.opcode == FS_TRANSPOSE || n.opcode == FS_CONCAT)
      FS_FAIL(FS_ERR_UNSUPPORTED, "node %d is not elementwise over the columns of [%d,%d]", m, gp.R, gp.C);
    gp.kind[m] = k;
    int lvl = 0;
    for (int i = 0; i < n.num_in; ++i) {
      Resolved r;
      if (g.flat_in[m][i] || !a.resolve(n.in[i], reduce ? KIND_FULL : k, false, &r)) FS_FAIL(FS_ERR_UNSUPPORTED, "node %d: operand %d", m, n.in[i]);
      if (r.literal) continue;
      if (r.kind != KIND_FULL && r.kind != KIND_ROWV) FS_FAIL(FS_ERR_UNSUPPORTED, "node %d: operand %d", m, n.in[i]);
      if (a.in_set[r.node]) {
        lvl = std::max(lvl, gp.level[r.node] + (g.nodes[r.node].opcode == FS_REDUCE_COL ? 1 : 0));
        continue;
      }
      if (a.in_set[g.root_of[r.node]]) FS_FAIL(FS_ERR_UNSUPPORTED, "node %d reads a view of a value of the same kernel", m);
      for (const ExtTensor& e : gp.ext_in)
        if (e.node == r.node && e.kind != r.kind) FS_FAIL(FS_ERR_UNSUPPORTED, "node %d is read in two ways", r.node);
      add_ext_in(gp, r.node, r.kind, g.nodes[r.node].dtype);
      gp.kind[r.node] = r.kind;
    }
    gp.level[m] = lvl;
    top = std::max(top, lvl);
    if (reduce) gp.col_reduces.push_back(m);
    bool leaves = g.output_index[m] >= 0 || read_by_others(m);
    for (int u : g.users[m]) leaves |= op_is_view(g.nodes[u].opcode);
    if (!leaves) continue;
    ExtTensor e;
    e.node = m, e.kind = k, e.dtype = n.dtype;
    gp.ext_out.push_back(e);
  }
  if (top == 0) FS_FAIL(FS_ERR_UNSUPPORTED, "nothing depends on a column reduction");
  if ((int)(gp.ext_in.size() + gp.ext_out.size()) > kMaxGroupTensors) FS_FAIL(FS_ERR_UNSUPPORTED, "group touches too many tensors");
  int arg = 0;
  for (ExtTensor& e : gp.ext_in) e.arg = arg++;
  for (ExtTensor& e : gp.ext_out) e.arg = arg++;
  auto bytes_of = [&](int id) { return (uint64_t)g.nodes[id].rows * g.nodes[id].cols * dtype_size(g.nodes[id].dtype); };
  for (ExtTensor& e : gp.ext_in) {
    e.streaming = e.kind == KIND_FULL && bytes_of(e.node) >= (g.nodes[g.root_of[e.node]].opcode == FS_INPUT && !read_by_others(g.root_of[e.node]) ? 2ull << 20 : kStreamBytes);
    if (e.kind == KIND_FULL) max_es = std::max(max_es, dtype_size(e.dtype));
    gp.min_hbm_bytes += bytes_of(e.node);
  }
  for (ExtTensor& e : gp.ext_out) {
    e.streaming = e.kind == KIND_FULL && bytes_of(e.node) >= (g.family_output[e.node] >= 0 && !read_by_others(e.node) ? 2ull << 20 : kStreamBytes);
    if (e.kind == KIND_FULL) max_es = std::max(max_es, dtype_size(e.dtype));
    gp.min_hbm_bytes += bytes_of(e.node);
  }
  if (max_es == 0) FS_FAIL(FS_ERR_UNSUPPORTED, "no [R,C] tensor");
  Schedule& s = gp.s;
  s.V = 16 / max_es;
  while ((int64_t)gp.C * max_es <= 32 ? gp.C % s.V != 0 : s.V > gp.C) s.V /= 2;
  s.NV = gp.C / s.V + (gp.C % s.V != 0);
  for (const ExtTensor& e : gp.ext_in)
    if (e.kind == KIND_FULL) dwords += std::max(1, s.V * dtype_size(e.dtype) / 4);
  // (32-bit offsets, also of the rows beyond the last one; accesses through a buffer descriptor start at whole words)
  if ((uint64_t)gp.R * gp.C * max_es > (1ull << 30)) FS_FAIL(FS_ERR_UNSUPPORTED, "tensors too large for the registers of the device");
  for (const auto* list : {&gp.ext_in, &gp.ext_out})
    for (const ExtTensor& e : *list)
      if (e.kind == KIND_FULL && gp.C % s.V != 0 && dtype_size(e.dtype) < 4) FS_FAIL(FS_ERR_UNSUPPORTED, "rows of %d columns of 2 bytes or less start inside a word", gp.C);
  const fs_status st = pick_join_shape(&gp, std::max(1, dwords), max_es);
  if (st != FS_OK) return st;
  s.ragged = gp.C % s.V != 0 || (int64_t)s.CT * s.L != s.NV;
  s.col_tiled = true;
  s.lds_bytes = s.lds_planned = ((s.L < 64 ? s.WG / 64 : s.G) + (int)gp.col_reduces.size()) * s.fold_width * 4 + (s.RB > 1 ? s.WG * 4 : 0) + 16;
  if (s.lds_bytes > opt.lds_budget) FS_FAIL(FS_ERR_LDS_BUDGET, "joined groups need %d bytes of LDS, budget is %d", s.lds_bytes, opt.lds_budget);
  if (s.RB > 1) {
    s.part_stride_floats = gp.col_reduces.size() * (size_t)s.fold_width * s.RB;
    // (a tile's counters share no cache line with another's; top: the last stage there can be)
    s.ticket_stride = join_counters(top + 1) + ((top + 1) * 2 * ((s.RB + 31) / 32) + 31) / 32 * 32;
    gp.n_tickets = s.ticket_stride * s.CT;
    gp.part_bytes = s.part_stride_floats * s.CT * 4;
  }
  gp.wait_ticks = wait_ticks(5000);
  if (s.WG >= 512 && tiles_share_lines(gp)) s.xcd_rows = 8;  // (smaller tensors: [4096,333] 10.0 against 10.2, [2000,1002] 10.4 against 10.6)
  return FS_OK;
}

// Folds of a few long rows that were kept out of the kernels beside them (worth_fusing) read the same tensors then, or values that they compute
// again from a number a row.  Where [R,C] values pass through memory between them instead, two or three launches follow each other in the
// place of one: column sums of a row softmax fp32 [400,8192] 25.4 us apart and 18.9 in one, [1900,2000] 25.9 and 17.1, of x less its row maximum [1500,3000]
// 27.0 and 14.3, [2000,3900] 33.9 and 18.6 (8192 columns that leave as well, [400,8192], 15.7 and 18.4).  Nor does a single fold pay that
// waits for numbers of the rows: column sum of a row softmax [300,8192] 11.2 and 12.4, [1000,2500] 13.9 and 11.8, [1900,2100] 19.3 and 14.8, two sums
// [300,8192] 12.1 and 17.6, [1300,2000] 14.7 and 16.7.  Such groups are formed again with their folds beside the row reductions, where that takes fewer
// kernels (one with five folds of [1000,513], beside a kernel of row reductions and a transpose, 38.1 us in two launches; two with three and two 50.8).
bool folds_exchange_rows(const Graph& g, const std::vector<std::vector<int>>& ordered, const std::vector<int>& group_of, const PlanOptions& opt) {
  if (ordered.size() < 2) return false;
  std::vector<GroupPlan> groups(ordered.size());
  std::map<int, size_t> stored_by;
  for (size_t k = 0; k < ordered.size(); ++k) {
    if (analyse_group(g, ordered[k], group_of, (int)k, opt, &groups[k]) != FS_OK) return false;  // (reported where the kernels are made)
    for (const ExtTensor& e : groups[k].ext_out) stored_by[e.node] = k;
  }
  auto folds = [&](size_t k) { return !groups[k].col_reduces.empty() && groups[k].R < 2048; };
  for (size_t k = 0; k < groups.size(); ++k)
    for (const ExtTensor& e : groups[k].ext_in) {
      auto it = stored_by.find(g.root_of[e.node]);
      if (it == stored_by.end() || it->second == k) continue;
      if (e.kind == KIND_FULL && (folds(k) || folds(it->second))) return true;
      if (e.kind == KIND_COLV && folds(k) && groups[k].col_reduces.size() == 1) return true;
    }
  return false;
}

// -------------------------------------------------------------------------------------------
// Groups that share a launch (Composite).
// -------------------------------------------------------------------------------------------
namespace {

struct Composer {
  const Graph& g;
  const std::vector<GroupPlan>& groups;
  const std::vector<int>& group_of;
  const PlanOptions& opt;
  std::map<int, int> stored_by;            // tensor in memory -> the group that stores it
  std::vector<std::set<int>> deps;         // groups whose results a group reads
  static constexpr uint64_t kSmall = 32ull << 20;  // bytes of a group whose launch, not its traffic, is what it costs (above, nothing was left to gain)
  static constexpr int kMaxTracks = 4, kMaxLds = 65536;

  Composer(const Graph& g_, const std::vector<GroupPlan>& groups_, const std::vector<int>& group_of_, const PlanOptions& o)
      : g(g_), groups(groups_), group_of(group_of_), opt(o), deps(groups_.size()) {
    for (size_t k = 0; k < groups.size(); ++k)
      for (const ExtTensor& e : groups[k].ext_out) stored_by[e.node] = (int)k;
    for (size_t k = 0; k < groups.size(); ++k)
      for (const ExtTensor& e : groups[k].ext_in) {
        auto it = stored_by.find(g.root_of[e.node]);
        if (it != stored_by.end() && it->second != (int)k) deps[k].insert(it->second);
      }
  }

  bool small(int k) const {
    const GroupPlan& p = groups[k];
    return !p.s.chunked && !p.s.split_rows && !p.s.resident && (p.s.U == 1 || !p.col_reduces.empty()) && !p.s.ahead && p.min_hbm_bytes <= kSmall;
  }

  // does workgroup b of `to` read of `from` only what workgroup b wrote, when both take the same rows?
  bool row_local(int from, int to) const {
    const GroupPlan &a = groups[from], &b = groups[to];
    if (a.R != b.R || !a.col_reduces.empty() || !b.col_reduces.empty()) return false;
    for (const ExtTensor& e : b.ext_in) {
      auto it = stored_by.find(g.root_of[e.node]);
      if (it == stored_by.end() || it->second != from) continue;
      if (it->first != e.node || (e.kind != KIND_COLV && e.kind != KIND_FULL)) return false;
      for (const ExtTensor& w : a.ext_out)
        if (w.node == e.node && (w.kind != e.kind || w.transposed || (e.kind == KIND_FULL && a.C != b.C))) return false;
    }
    return true;
  }

  // group k with L lanes a row (0: its own) and WG lanes a workgroup, one trip to a workgroup
  bool plan(int k, int L, int WG, bool chain, GroupPlan* out) const {
    if (!groups[k].col_reduces.empty()) {  // as it is: partials and counters are laid out for it
      *out = groups[k];
      return L <= 0 && out->s.WG == WG;
    }
    const Schedule& was = groups[k].s;
    if (L <= 0) L = was.L;
    if (L == was.L && WG == was.WG && was.min_waves == 0) {
      *out = groups[k];
    } else {
      PlanOptions o = opt;
      o.hint = fs_sched_hint{L, WG, 0, 0};
      o.has_hint = true;
      o.fill_lanes = chain;
      o.keep_flat = groups[k].flat > 0;
      if (analyse_group(g, groups[k].members, group_of, k, o, out) != FS_OK) return false;
    }
    const Schedule& s = out->s;
    return s.WG == WG && s.L == L && s.V * s.spread == was.V && s.grid == s.n_iters && s.U == 1 && !s.chunked && !s.resident && !s.split_rows && !s.ahead && s.tile_transpose >= was.tile_transpose;
  }

  // plans for all tracks with a common workgroup; false where they do not agree or do not fit
  bool fit(Composite* c) const {
    // the largest workgroup among them, or that of a column fold, whose partials are laid out for it
    c->WG = 0;
    bool folds = false;
    for (const auto& t : c->tracks)
      for (int k : t) {
        const bool f = !groups[k].col_reduces.empty();
        if (f > folds || (f == folds && groups[k].s.WG > c->WG)) c->WG = groups[k].s.WG;
        folds |= f;
      }
    c->plans.assign(c->tracks.size(), {});
    c->blocks.assign(c->tracks.size(), 0);
    int pointers = 0, lds = 0, parts = 0;
    for (size_t t = 0; t < c->tracks.size(); ++t) {
      int L = 0;
      for (int k : c->tracks[t]) L = std::max(L, groups[k].s.L);
      for (int k : c->tracks[t]) {
        GroupPlan p;
        const bool chain = c->tracks[t].size() > 1;
        if (!plan(k, chain ? L : 0, c->WG, chain, &p)) return false;
        // (a workgroup of column tiles has part of its rows: what the next group reads of them others have written)
        if (chain && (p.s.CT > 1 || p.s.col_tiled || p.s.tiled_transpose)) return false;
        if (c->blocks[t] != 0 && p.s.grid != c->blocks[t]) return false;
        c->blocks[t] = p.s.grid;
        pointers += (int)(p.ext_in.size() + p.ext_out.size());
        lds += p.s.lds_bytes;
        c->plans[t].push_back(std::move(p));
        ++parts;
      }
    }
    return pointers <= kMaxCompositePointers && parts <= kMaxCompositeGroups && lds <= std::min(kMaxLds, opt.lds_budget);
  }
};

void replace_all(std::string* s, const std::string& from, const std::string& to) {
  for (size_t p = 0; (p = s->find(from, p)) != std::string::npos; p += to.size()) s->replace(p, from.size(), to);
}

// What passes between the groups of a chain.  Per-row results stay in registers: loads that are asked for after stores wait for them, so a
// group that reads the last one's results from memory waits until all of them are written.  Where a group needs nothing else from
// those before it, there is no barrier, and its other tensors are asked for first of all (they may take kAsked registers).  The same
// random DAG of 200 ops, rows x width: [512,256] 22.7 -> 20.5 us, [512,128] 20.5 -> 17.8, [333,77] 22.7 -> 18.7, [64,1024] 28.4 -> 24.7, [2048,128]
// 25.6 -> 24.6.
void link_chain(std::vector<GroupPlan>* parts, std::string* fields) {
  constexpr int kAsked = 64;
  int asked = 0;
  for (size_t k = 1; k < parts->size(); ++k) {
    GroupPlan& p = (*parts)[k];
    std::map<int, size_t> from;  // results of the groups before -> their group
    bool linked = true;
    for (const ExtTensor& e : p.ext_in)
      for (size_t b = 0; b < k; ++b)
        for (const ExtTensor& w : (*parts)[b].ext_out)
          if (w.node == e.node) {
            from[e.node] = b;
            linked &= e.kind == KIND_COLV && w.kind == KIND_COLV && e.dtype == FS_F32 && w.dtype == FS_F32;
            for (const ExtTensor& o : p.ext_in) linked &= o.node != e.node || o.kind == KIND_COLV;
          }
    if (!linked) continue;
    p.s.stage_rowv = false;
    p.linked = true;
    p.source.clear();
    for (const ExtTensor& e : p.ext_in) {
      const std::string name = "g" + std::to_string(k) + "_" + std::to_string(e.node);
      auto it = from.find(e.node);
      const int regs = e.kind == KIND_COLV ? 1 : p.s.E;
      if (p.comes.count(e.node)) continue;
      int uses = 0;  // (a tensor that is read in two ways comes from memory)
      for (const ExtTensor& o : p.ext_in) uses += o.node == e.node;
      if (it != from.end()) {
        GroupPlan& b = (*parts)[it->second];
        if (!b.leaves.count(e.node)) {
          b.leaves[e.node] = name;
          b.source.clear();
          *fields += " float " + name + ";";
        }
        p.comes[e.node] = b.leaves[e.node];
      } else if ((e.kind == KIND_COLV || e.kind == KIND_FULL || e.kind == KIND_ROWV) && uses == 1 && asked + regs <= kAsked) {
        asked += regs;
        p.comes[e.node] = name;
        p.asked.insert(e.node);
        *fields += " float " + name + (e.kind == KIND_COLV ? ";" : "[" + std::to_string(p.s.E) + "];");
      }
    }
  }
}

// the kernels of a composite become functions of one kernel
bool generate_composite(const Graph& g, Composite* c) {
  std::vector<std::string> fields(c->tracks.size());
  for (size_t t = 0; t < c->tracks.size(); ++t) link_chain(&c->plans[t], &fields[t]);
  for (size_t t = 0; t < c->tracks.size(); ++t)
    for (size_t k = 0; k < c->plans[t].size(); ++k)
      if (c->plans[t][k].source.empty() && generate_kernel(g, &c->plans[t][k], c->tracks[t][k]) != FS_OK) return false;
  std::string text, body;
  std::set<std::string> seen;
  int total = 0;
  std::string args;
  bool passes = false;  // (one form for all tracks: a group's functions are defined once, whichever tracks it is in)
  for (const std::string& f : fields) passes |= !f.empty();
  for (size_t t = 0; t < c->tracks.size(); ++t) {
    body += std::string("  ") + (t + 1 < c->tracks.size() ? "if (block < " + std::to_string(c->blocks[t]) + ") {\n" : "{\n");
    int xcd_rows = 0;
    for (const GroupPlan& p : c->plans[t]) xcd_rows = xcd_rows == 0 || p.s.xcd_rows == 0 ? std::max(xcd_rows, p.s.xcd_rows) : std::min(xcd_rows, p.s.xcd_rows);
    const std::string place = xcd_rows ? "fs_xcd_place<" + std::to_string(xcd_rows) + ">(block, " + std::to_string(c->blocks[t]) + ")" : "block";
    if (passes) {
      body += "    struct {" + fields[t] + " } x;\n";
      for (size_t k = 1; k < c->plans[t].size(); ++k)
        if (!c->plans[t][k].asked.empty()) body += "    " + c->plans[t][k].kernel_name + "_ask(a.g" + std::to_string(total + (int)k) + ", " + place + ", x);\n";
    }
    for (size_t k = 0; k < c->plans[t].size(); ++k) {
      const GroupPlan& p = c->plans[t][k];
      const std::string field = "g" + std::to_string(total++), n = p.kernel_name;
      // (a kernel that folds columns, alone in its track, places its workgroups itself: their partials lie by block, as they do in a launch of its own)
      const bool folds = !p.col_reduces.empty();
      if (seen.insert(n).second) {
        std::string src = p.source;
        const size_t a = src.find("extern \"C\" __global__"), b = src.find("{\n", a);
        src.replace(a, b - a, (passes ? "template <class X> FS_DEV void " : "FS_DEV void ") + n + "_rows(const " + n + "_args& a, const int fs_block, const int fs_blocks" + (passes ? ", X& x) " : ") "));
        replace_all(&src, "struct " + n + "_args", "struct " + n + "_part_args");
        replace_all(&src, "const " + n + "_args&", "const " + n + "_part_args&");
        replace_all(&src, n + "_kinds", n + "_part_kinds");
        if (p.s.xcd_rows && !folds) replace_all(&src, "fs_xcd_place<" + std::to_string(p.s.xcd_rows) + ">((int)blockIdx.x, (int)gridDim.x)", "fs_block");
        replace_all(&src, "blockIdx.x", "fs_block");
        replace_all(&src, "gridDim.x", "fs_blocks");
        text += src;
      }
      args += "  " + n + "_part_args " + field + ";\n";
      // (what a workgroup wrote before the barrier it reads after it: the vector cache of a compute unit writes through)
      if (k > 0 && !p.linked) body += "    __syncthreads();\n";
      body += "    " + n + "_rows(a." + field + ", " + (folds ? "block" : place) + ", " + std::to_string(c->blocks[t]) + (passes ? ", x" : "") + ");\n";
    }
    body += "    return;\n  }\n";
    if (t + 1 < c->tracks.size()) body += "  block -= " + std::to_string(c->blocks[t]) + ";\n";
  }
  uint64_t h = 1469598103934665603ull;
  for (unsigned char ch : text + body) h = (h ^ ch) * 1099511628211ull;
  char nm[64];
  snprintf(nm, sizeof(nm), "fs_c_%016llx", (unsigned long long)h);
  c->kernel_name = nm;
  std::string head = "// one launch:";
  for (size_t t = 0; t < c->tracks.size(); ++t) {
    head += t ? " | groups" : " groups";
    for (int k : c->tracks[t]) head += " " + std::to_string(k);
    head += " on " + std::to_string(c->blocks[t]) + " workgroups";
  }
  // (in a namespace: another composite of the plan may hold the same group's functions)
  c->source = head + "\nnamespace " + c->kernel_name + "_parts {\n" + text + "struct " + c->kernel_name + "_args {\n" + args + "};\nextern \"C\" __global__ void __launch_bounds__(" + std::to_string(c->WG) + ") " + c->kernel_name + "(const " +
              c->kernel_name + "_args a) {\n  int block = (int)blockIdx.x;\n" + body + "}\n}\n";
  return true;
}

}  // namespace

// Launch-bound groups cost what a launch costs, whatever they move: a kernel that loads a row, computes and stores little takes
// 2.6-3 us.  A chain of groups over the same rows, of which each reads only what the same rows of the others wrote, runs as one
// kernel: a workgroup takes its rows through all of them (link_chain).  Chains and single groups that do not depend
// on each other run side by side on workgroups of their own.
void compose_groups(const Graph& g, const std::vector<GroupPlan>& groups, const std::vector<int>& group_of, const std::vector<std::pair<int, int>>& joined,
                    const PlanOptions& opt, bool may_share, std::vector<Composite>* composites, std::vector<LaunchItem>* launches) {
  composites->clear();
  launches->clear();
  Composer c(g, groups, group_of, opt);
  const int n = (int)groups.size();
  // the launches in order, as tracks of groups (a joined run is one that nothing joins)
  struct Item {
    Composite comp;
    int joined = -1;
    std::set<int> holds;
  };
  std::vector<Item> items;
  for (int k = 0; k < n; ++k) {
    Item it;
    for (size_t j = 0; j < joined.size(); ++j)
      if (joined[j].first == k) it.joined = (int)j;
    const int last = it.joined >= 0 ? k + joined[it.joined].second - 1 : k;
    for (int m = k; m <= last; ++m) it.holds.insert(m);
    if (it.joined < 0) it.comp.tracks = {{k}};
    items.push_back(it);
    k = last;
  }
  auto open = [&](const Item& it) { return may_share && it.joined < 0 && c.small(*it.holds.begin()); };
  auto ready = [&](const std::set<int>& holds, size_t before, const std::set<int>& besides) {  // everything they read is launched before, or in `besides` or `holds`
    std::set<int> done(besides);
    done.insert(holds.begin(), holds.end());
    for (size_t i = 0; i < before; ++i) done.insert(items[i].holds.begin(), items[i].holds.end());
    for (int k : holds)
      for (int d : c.deps[k])
        if (!done.count(d)) return false;
    return true;
  };
  auto take = [&](size_t into, size_t from, const Composite& comp) {
    items[into].comp = comp;
    items[into].holds.insert(items[from].holds.begin(), items[from].holds.end());
    items.erase(items.begin() + (long)from);
  };
  for (int pass = 0; pass < 2; ++pass)  // chains first, then what runs beside them
    for (size_t i = 0; i < items.size(); ++i) {
      if (!open(items[i])) continue;
      for (size_t j = i + 1; j < items.size();) {
        bool ok = open(items[j]) && (pass == 1 || items[j].comp.tracks.size() + items[j].comp.tracks[0].size() == 2);
        Composite trial = items[i].comp;
        if (ok && pass == 0) {  // at the end of the chain: of its groups it reads rows only, everything else is there already
          const int k = *items[j].holds.begin();
          bool reads = false;
          for (int d : c.deps[k])
            if (items[i].holds.count(d)) reads = true, ok &= c.row_local(d, k);
          ok &= reads && ready(items[j].holds, i, items[i].holds);
          if (ok) trial.tracks[0].push_back(k);
        } else if (ok) {
          ok = ready(items[j].holds, i, std::set<int>()) && trial.tracks.size() < Composer::kMaxTracks && items[j].comp.tracks.size() == 1;
          if (ok) trial.tracks.push_back(items[j].comp.tracks[0]);
        }
        if (ok && c.fit(&trial)) take(i, j, trial);
        else ++j;
      }
    }
  for (const Item& it : items) {
    LaunchItem l;
    if (it.joined >= 0) l.kind = LaunchItem::JOINED, l.index = it.joined;
    else if (it.holds.size() == 1) l.kind = LaunchItem::GROUP, l.index = *it.holds.begin();
    else {
      l.kind = LaunchItem::COMPOSITE, l.index = (int)composites->size();
      composites->push_back(it.comp);
      if (!generate_composite(g, &composites->back())) {  // (its groups one by one, in their order)
        composites->pop_back();
        for (int k : it.holds) launches->push_back({LaunchItem::GROUP, k});
        continue;
      }
    }
    launches->push_back(l);
  }
}

void work_span(const Graph& g, std::vector<int>* span) {
  PlanOptions opt;
  Former f(g, opt);
  f.mark_live();
  *span = f.spans();
}

}  // namespace fs
