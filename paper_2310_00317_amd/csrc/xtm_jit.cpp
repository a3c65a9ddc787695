// xtm_jit.cpp -- per-line tracking kernels generated and compiled at run time.
//
// The paper's tracker assembles and compiles one kernel that tracks the whole
// beam line.  On gfx950 the reason to do so is sharper than on a CPU: with
// one particle per lane and often fewer than two waves per SIMD, a generic
// element interpreter spends more issue slots on scalar dispatch (type
// decode, compare tree, loop control, register shuffling between switch arms)
// than on the FP64 maps.  Here the element-type sequence is cut into cells of
// a fixed period; each distinct cell signature ("kind") becomes one
// straight-line block of map calls with compile-time parameter offsets, and
// the kernel loops over the cells of a turn with one scalar branch per cell.
// Element parameters stay data (one array, read with scalar loads), so all
// lattices with the same structure share one compiled kernel.
#include <hip/hip_runtime.h>
#include <hip/hiprtc.h>

#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <sstream>
#include <string>
#include <vector>

#include "xtm_internal.h"

namespace xtm {

static const char* kMapsSource =
#include "xtm_maps_src.inc"
    ;

namespace {

struct Compiled {
  hipModule_t module = nullptr;
  hipFunction_t fn = nullptr;
  std::string error;
};

std::mutex g_mu;
std::map<std::string, Compiled> g_cache;  // schedule + generated source -> compiled kernel

uint32_t sig_of(uint64_t h) { return (uint32_t)(h & 0xffffu); }  // kernel type | order << 8
// added to the signature of a multipole whose parameters end in the reciprocal
// of its radiation length (straight cells)
constexpr uint32_t kRecip = 1u << 16;

struct Decomp {
  std::vector<std::vector<uint32_t>> kinds;  // element signatures of each kind
  std::vector<int32_t> cell_kind;            // kind of each cell, in line order
  std::vector<int32_t> cell_start;           // first element index of each cell
};

// Cover the line with cells: a repeating unit U of P elements wherever it
// matches, and the stretches in between ("gaps", e.g. a lone RF cavity or a
// cell whose sextupole slot holds a cavity) as further kinds, split into
// pieces of at most max_unit elements.  Among all units (P <= max_unit,
// every phase) keep the cover with the fewest cells whose distinct kinds
// need at most max_code elements of generated code.
constexpr int kMaxUnit = 24;
constexpr int kMaxCode = 48;
// the long-cell forms
constexpr int kLongUnit = 40;
constexpr int kLongCode = 64;
// parameter words between two settled points of a straight cell, at least:
// every drift of the FODO and DA rings (12 and 23 words apart), every second
// or third of a ring of sliced magnets (5 to 8 words a slice).  More between
// them costs the first two registers (DA ring, 40,000 particles: 4.05e11
// passes/s settled at every drift, 3.79e11 at every second, 3.38e11 at none),
// less costs the last overlap (thick ring, 30,000: 3.48e11 at every drift,
// 3.65e11-3.80e11 at every second to fourth)
constexpr int32_t kSettleWords = 12;
// parameter words that a cell of the wide form holds in scalar registers (two
// a word, of 102): an element's words are read further ahead of it only while
// those of the elements in between fit, else at the element itself.  Without
// the limit the registers are spilled in the middle of a cell that has several
// high-order multipoles in a row (three of order 10 and a drift: 1,145 lane moves
// among 3,051 instructions, with it 189 among 2,071); a batch of rings with two
// of order 10 in a row takes the same time either way
constexpr int32_t kScalarWords = 24;
// cells ahead of the tracking wave that the recording kernel's other wave loads
constexpr int32_t kAhead = 4;

// (Longest units first: a unit that cannot beat the best cover so far, or that
// needs too much code, is given up at once, which leaves a few full scans of the
// line: 20,000 elements in cells of 10, 25 ms -> 5 ms.)
bool decompose(const std::vector<uint32_t>& sig, Decomp* out, int32_t max_unit = kMaxUnit,
               int32_t max_code = kMaxCode) {
  const int32_t E = (int32_t)sig.size();
  if (E == 0) return false;
  size_t best_cells = 0;
  int32_t best_code = 0;
  for (int32_t P = std::min(max_unit, E); P >= 1; --P) {
    bool best_has_p = false;  // the first phase of a unit length wins ties
    for (int32_t o = 0; o < P && o + P <= E; ++o) {
      const uint32_t* U = &sig[o];
      std::map<std::vector<uint32_t>, int32_t> kinds;
      kinds.emplace(std::vector<uint32_t>(U, U + P), 0);
      int32_t code = P;
      Decomp d;
      d.kinds.push_back(std::vector<uint32_t>(U, U + P));
      bool ok = code <= max_code;
      auto add = [&](int32_t start, int32_t len) {
        std::vector<uint32_t> t(sig.begin() + start, sig.begin() + start + len);
        auto it = kinds.find(t);
        if (it == kinds.end()) {
          code += len;
          it = kinds.emplace(t, (int32_t)d.kinds.size()).first;
          d.kinds.push_back(t);
        }
        d.cell_kind.push_back(it->second);
        d.cell_start.push_back(start);
        ok &= code <= max_code;
      };
      int32_t i = 0, gap = -1;
      while (i < E && ok) {
        // no cell is longer than max_unit
        if (best_cells &&
            d.cell_kind.size() + (size_t)(E - (gap >= 0 ? gap : i) + max_unit - 1) / max_unit >
                best_cells) {
          ok = false;
          break;
        }
        if (i + P <= E && std::memcmp(&sig[i], U, P * sizeof(uint32_t)) == 0) {
          if (gap >= 0) add(gap, i - gap), gap = -1;
          d.cell_kind.push_back(0);
          d.cell_start.push_back(i);
          i += P;
        } else {
          if (gap < 0) gap = i;
          ++i;
          if (i - gap == max_unit) add(gap, max_unit), gap = -1;  // a full piece of the gap
        }
      }
      if (ok && gap >= 0) add(gap, E - gap);
      if (!ok) continue;
      const size_t cells = d.cell_kind.size();
      if (best_cells == 0 || cells < best_cells ||
          (cells == best_cells && (code < best_code || (code == best_code && !best_has_p)))) {
        best_cells = cells;
        best_code = code;
        best_has_p = true;
        *out = d;
      }
    }
  }
  return best_cells > 0;
}

int32_t n_words(uint32_t s) {
  const uint32_t kt = s & 0xffu, order = (s >> 8) & 0xffu;
  switch (kt) {
    case K_DRIFT: case K_DRIFT_EXP: case K_AP_CIRC: return 1;
    case K_MULT: return 2 * ((int32_t)order + 1);
    case K_MULT_CURV: return 2 * ((int32_t)order + 1) + 3 + ((s & kRecip) ? 1 : 0);
    case K_MULT_LR: return 2 * ((int32_t)order + 1) + 1 + ((s & kRecip) ? 1 : 0);
    case K_RF: return 3;
    case K_SHIFT: case K_SROT: case K_AP_ELL: return 2;
    case K_AP_RECT: return 4;
    default: return 0;
  }
}

// C++ statement applying one element whose parameters are P[0..] where P is
// the expression `arr` (an LDS pointer "p + o" or a local array name); `j` is
// the expression of its position in the cell (the loss code is e0 + j).
// Loss handling (`mode`): kSaveAtLoss stores a failing lane's entry
// coordinates at the element; kMarkOnly only records the loss code (the cell
// is replayed for lanes lost in it, see generate); kReplay applies the map
// alone (the replay itself).
// kFlag: no branch and no store; a failing test, or operands the drift's short
// sequences do not serve, set `bad`.
// kTest: the generic drift, and a loss test's result in `ok` with the state a
// lost particle takes in `ls`.
// kFlagScalar, kTestScalar: as kFlag and kTest from the wide form's parameters
// (wide_words), the former's in scalar registers.
enum EmitMode {
  kSaveAtLoss = 0, kMarkOnly = 1, kReplay = 2, kFlag = 4, kTest = 5, kFlagScalar = 6,
  kTestScalar = 7
};

// batched: for a kernel that serves a batch of lattice variants.  rf_by_vector:
// a cavity's series reads its table through vector registers.
std::string emit(uint32_t s, const std::string& arr, const std::string& j, bool far_rf,
                 EmitMode mode, bool batched = false, bool rf_by_vector = false) {
  const uint32_t kt = s & 0xffu, order = (s >> 8) & 0xffu;
  auto P = [&](int32_t m) { return "(" + arr + ")[" + std::to_string(m) + "]"; };
  const bool flag = mode == kFlag || mode == kFlagScalar;
  const bool negated = mode == kFlagScalar || mode == kTestScalar;
  // multipole's second parameter (a batch's slot partition takes scalar registers)
  const std::string sc = !negated ? "" : batched ? ", 2" : ", 1";
  // the radiation step of a multipole whose radiation length is word m
  auto radiation = [&](int32_t m) {
    return flag && (s & kRecip)
               ? "RADF(kx, ky, " + P(m) + ", " + P(m + 1) + ", " + j + ");"
               : "RAD(kx, ky, " + P(m) + ", " + j + ");";
  };
  std::ostringstream c;
  switch (kt) {
    case K_DRIFT: {
      // the drift record's order: the length's class for the short sequences
      const std::string any = std::to_string(order);
      if (mode == kReplay)
        c << "(void)xtmm::drift_exact(q, " << P(0) << ", " << any << ");";
      else if (flag)
        c << "xtmm::drift_flag<" << (mode == kFlagScalar ? "true" : "false") << ">(q, " << P(0)
          << ", " << any << ", a_min, bad);";
      else if (mode == kTest || mode == kTestScalar)
        c << "{ const xtmm::DriftIn d_ = xtmm::drift_in(q); double lp_, dq_; "
          << "xtmm::drift_generic(" << (negated ? "-" : "") << P(0) << ", d_, lp_, dq_); "
          << "xtmm::drift_apply(q, lp_, dq_); ok = d_.pz2 > 0.0; ls = -1; }";
      else if (mode == kMarkOnly)
        c << "xtmm::mark(xtmm::drift_exact(q, " << P(0) << ", " << any << "), code, st, e0 + "
          << j << ", -1);";
      else
        // one rare branch per drift: operands outside the window take the
        // generic operations, and a lane lost here stores its entry state
        c << "{ const xtmm::DriftIn d_ = xtmm::drift_in(q); double lp_, dq_; bool f_; "
          << "xtmm::drift_quotients(" << P(0) << ", d_, " << any << ", lp_, dq_, f_); "
          << "if (!f_) { if (!(d_.pz2 > 0.0) && live) { SAVE(); code = e0 + " << j
          << "; st = -1; live = false; } xtmm::drift_generic(" << P(0)
          << ", d_, lp_, dq_); } xtmm::drift_apply(q, lp_, dq_); }";
      break;
    }
    case K_DRIFT_EXP:
      c << "xtmm::drift_expanded(q, " << P(0) << ");";
      break;
    case K_MULT:
      c << "{ double kx, ky; xtmm::multipole<" << order << sc << ">(q, " << arr << ", kx, ky); }";
      break;
    case K_MULT_CURV: {
      const int32_t v = 2 * ((int32_t)order + 1);
      c << "{ double kx, ky; xtmm::multipole<" << order << sc << ">(q, " << arr
        << ", kx, ky); "
        << (flag && (s & kRecip) ? "xtmm::curvature_flag(q, " : "xtmm::curvature(q, ") << P(v)
        << ", " << P(v + 1) << ", " << P(v + 2);
      if (flag && (s & kRecip)) c << ", " << P(v + 3) << ", bad";
      c << "); " << radiation(v + 2) << " }";
      break;
    }
    case K_MULT_LR: {
      const int32_t v = 2 * ((int32_t)order + 1);
      c << "{ double kx, ky; xtmm::multipole<" << order << sc << ">(q, " << arr
        << ", kx, ky); " << radiation(v) << " }";
      break;
    }
    case K_RF:
      c << (far_rf ? "xtmm::rf_far(q, " : rf_by_vector ? "xtmm::rf<xtmm::kByVector>(q, " : "xtmm::rf(q, ")
        << P(0) << ", " << P(1) << ", " << P(2) << ", beta0, two_over_beta0);";
      if (flag)
        c << " bad |= !xtmm::drift_range(q); "
             "if (__builtin_bit_cast(unsigned long long, q.u) != 0) a_min = xtmm::kDriftMin;";
      break;
    case K_SHIFT:
      c << "xtmm::xyshift(q, " << P(0) << ", " << P(1) << ");";
      break;
    case K_SROT:
      c << "xtmm::srotation(q, " << P(0) << ", " << P(1) << ");";
      break;
    case K_AP_CIRC:
    case K_AP_ELL:
    case K_AP_RECT: {
      if (mode == kReplay) break;  // a test, no change of coordinates
      std::string test;
      if (kt == K_AP_CIRC) test = "xtmm::in_circle(q, " + P(0) + ")";
      else if (kt == K_AP_ELL) test = "xtmm::in_ellipse(q, " + P(0) + ", " + P(1) + ")";
      else test = "xtmm::in_rect(q, " + P(0) + ", " + P(1) + ", " + P(2) + ", " + P(3) + ")";
      if (flag) {
        c << "bad |= !" << test << ";";
        break;
      }
      if (mode == kTest || mode == kTestScalar) {
        c << "ok = " << test << "; ls = 0;";
        break;
      }
      c << "{ const bool ok = " << test << "; ";
      if (mode == kSaveAtLoss)
        c << "if (!ok && live) { SAVE(); code = e0 + " << j << "; st = 0; live = false; } }";
      else
        c << "xtmm::mark(ok, code, st, e0 + " << j << ", 0); }";
      break;
    }
    default:
      break;  // marker
  }
  return c.str();
}

int32_t kind_words(const std::vector<uint32_t>& k) {
  int32_t w = 0;
  for (uint32_t s : k) w += n_words(s);
  return w;
}

// Constant tables of a second, element by element pass through a cell: per
// kind its first entry; per entry its element's signature (the index in
// `sigs`, the line's distinct ones) and parameter offset.
std::string replay_tables(const Decomp& d, std::vector<uint32_t>* sigs) {
  std::ostringstream kf, es, eo;
  int32_t n = 0;
  for (const auto& k : d.kinds) {
    kf << n << ", ";
    int32_t o = 0;
    for (uint32_t e : k) {
      size_t g = 0;
      while (g < sigs->size() && (*sigs)[g] != e) ++g;
      if (g == sigs->size()) sigs->push_back(e);
      es << g << ", ";
      eo << o << ", ";
      o += n_words(e);
      ++n;
    }
  }
  kf << n;
  return "__constant__ int kind_first[] = {" + kf.str() + "};\n"
         "__constant__ int elem_sig[] = {" + es.str() + "};\n"
         "__constant__ int elem_off[] = {" + eo.str() + "};\n";
}

// For element m of a kind: the element before whose arithmetic its words are
// read, m - 1, or, for an element of many words (a high-order multipole) after
// a short test or frame change, m - 2: the aperture's few operations would not
// cover the multipole's reads.  (Reading a drift's one word that early costs
// the saturated rings more registers than it saves.)
std::vector<size_t> reads_ahead(const std::vector<uint32_t>& kd) {
  std::vector<size_t> before(kd.size(), 0);
  for (size_t m = 1; m < kd.size(); ++m) {
    const uint32_t kp = kd[m - 1] & 0xffu;
    const bool short_prev = kp == K_AP_CIRC || kp == K_AP_ELL || kp == K_AP_RECT ||
                            kp == K_SHIFT || kp == K_SROT || kp == K_MARKER;
    before[m] = (short_prev && m >= 2 && n_words(kd[m]) >= 8) ? m - 2 : m - 1;
  }
  return before;
}

// Registers of an element's parameters (element j, first word `off`), read in
// one group.
void read_words(std::ostringstream& s, uint32_t sig, size_t j, int32_t off) {
  const int32_t nw = n_words(sig);
  if (nw == 0) return;
  s << "        double w" << j << "[" << nw << "];\n"
    << "#pragma unroll\n"
    << "        for (int m = 0; m < " << nw << "; ++m) w" << j << "[m] = p[" << off << " + m];\n";
}

// The statements of one straight cell.  A drift starts from settled momenta,
// and the reads that follow stay behind this point (both pass through an empty
// register constraint); in between, the arithmetic may move.  at(j): a
// statement before element j, and whether the element is left out.
template <typename At>
void straight_cell(std::ostringstream& s, const std::vector<uint32_t>& kd, bool scalar,
                   bool batched, At at) {
  std::vector<int32_t> off(kd.size() + 1, 0);
  for (size_t j = 0; j < kd.size(); ++j) off[j + 1] = off[j] + n_words(kd[j]);
  std::vector<size_t> before = reads_ahead(kd);
  for (size_t m = 1; scalar && m < kd.size(); ++m)
    for (; before[m] < m; ++before[m]) {
      int32_t held = 0;
      for (size_t k = before[m]; k <= m; ++k) held += n_words(kd[k]);
      if (held <= kScalarWords) break;
    }
  // a cavity's table is 14 words: beside high-order multipoles it does not fit.
  // (200 cells of a cavity, drifts and quadrupoles, 1M particles, 20 turns: 29.2
  // ms by scalar registers, 29.9 ms by vector registers; a cavity between
  // multipoles of order 10: 1,130 lane moves in a cell against 79.)
  int32_t longest = 0;
  for (uint32_t e : kd) longest = std::max(longest, n_words(e));
  const bool rf_by_vector = scalar && longest + 14 > kScalarWords;
  if (!kd.empty()) read_words(s, kd[0], 0, 0);
  int32_t since = 0;  // parameter words since the last settled point
  for (size_t j = 0; j < kd.size(); ++j) {
    const uint32_t kt = kd[j] & 0xffu;
    const bool settle = (kt == K_DRIFT || kt == K_DRIFT_EXP) && since >= kSettleWords;
    if (settle) since = 0;
    since += n_words(kd[j]);
    s << "        asm volatile(\"\" : \"+" << (scalar ? "s" : "v") << "\"(p)"
      << (settle ? ", \"+v\"(q.px), \"+v\"(q.py), \"+v\"(q.zeta)" : "") << ");\n";
    for (size_t m = j + 1; m < kd.size() && m <= j + 2; ++m)
      if (before[m] == j) read_words(s, kd[m], m, off[m]);
    if (j > 0 && before[j] == j) read_words(s, kd[j], j, off[j]);
    const std::pair<std::string, bool> extra = at(j);
    if (!extra.first.empty()) s << "        " << extra.first << "\n";
    if (extra.second) continue;
    const std::string arr =
        n_words(kd[j]) > 0 ? "w" + std::to_string(j) : "p + " + std::to_string(off[j]);
    const std::string stmt =
        emit(kd[j], arr, std::to_string(j), false, scalar ? kFlagScalar : kFlag, batched,
             rf_by_vector);
    if (!stmt.empty()) s << "        " << stmt << "\n";
  }
}

// The smallest drift numerator that a lane's short sequences serve, as the
// kernel starts; axis: the line keeps the reference particle on the axis.
const char* a_min_init(bool axis) {
  return axis ? "xtmm::on_axis(q) ? 0.0 : xtmm::kDriftMin" : "xtmm::kDriftMin";
}

// Generated kernel.  Per cell the workgroup holds the cell's parameters in
// one of two LDS slots: while the waves compute cell g from slot g&1, each
// thread has already loaded its share of cell g+1's parameters from global
// memory and writes it to the other slot before the cell barrier.  Element
// code then reads its parameters as broadcast LDS reads at compile-time
// offsets.
std::string generate(const Decomp& d, int32_t style, bool batched, int32_t rad_form,
                     bool flagged, bool scalar, bool axis) {
  int32_t maxw = 1;
  for (const auto& k : d.kinds) maxw = std::max(maxw, kind_words(k));
  // the lanes of a workgroup share one LDS slot pair, filled by all of them
  // and fenced by workgroup barriers (line_block: 256 lanes, or one wave)
  const int32_t lanes = line_block(style);
  // how element code reads its parameters from the slot (line_fetch):
  // 0 = at each use (the compiler interleaves the reads with the arithmetic),
  // 1 = all of an element's words in one group before its arithmetic,
  // 2 = the next element's group issued before the current element's
  //     arithmetic, so the read latency overlaps one element of work
  const int32_t fetch = line_fetch(style);
  // loss handling: at each loss test (a divergent store per test), or once
  // per cell (line_deferred: the tests only record the loss code; lanes lost
  // in the cell replay it afterwards)
  const bool deferred = line_deferred(style);
  // (flagged) or once per cell without recording which test failed: the
  // cell is one straight run of arithmetic, and lanes that failed some test
  // in it, or met a drift outside the short sequences' window, go through it
  // again from its entry with each test where it belongs.
  //   What bounds it: a wave alone on its SIMD waits on its own dependent
  //   operations (a drift is 17 of them from momenta to positions), and a
  //   branch per drift and per aperture kept the next element's operations,
  //   and the drift's quotient for zeta that nothing waits for, from filling
  //   those waits.  Without the branches (and with 38 instead of 40 operations
  //   a drift, see drift_flag): FODO ring, 1,000 particles, 47 -> 38 us per
  //   turn; DA ring, 40,000 particles, 3.5e11 -> 4.05e11 passes/s; sliced
  //   ring, 30,000 particles, 3.1e11 -> 3.6e11.
  //   The register constraints below hold the compiler to one drift's work in
  //   flight: left alone it keeps every pending quotient and parameter of the
  //   cell in registers (over 300, one wave per SIMD, 1M particles of the
  //   FODO ring 12.1 ms instead of 8.4 ms).
  // The wide form (`scalar`): the parameters come through scalar loads into
  // scalar registers, which a fused multiply-add takes as its addend (kept
  // negated, see xtmm::addend and wide_words).  With several waves per SIMD the
  // broadcast reads of LDS bound the rings of high order multipoles (an order-10
  // multipole reads 11 x 16 bytes for 64 lanes and computes 42 operations), and
  // their registers kept the waves at two per SIMD.  In scalar registers they cost
  // no LDS reads and leave three or four waves (93-122 vector registers on the
  // FODO, DA and errored rings); what they cost is scalar registers, of which the
  // loop's own are spilled (44-90 of them; in the hot cell 41 lane moves of 1,487
  // instructions on the errored ring, none on the other two).  Error seeds of the FODO ring, 1M particles: 6.1e11
  // -> 8.8e11 passes/s; DA ring, 131,072: 6.3e11 -> 7.8e11; FODO ring, 1M:
  // 1.95e12 -> 2.0e12.  A lone wave waits longer for scalar loads (one every
  // 64 bytes) than for LDS: DA ring, 40,000 particles, 3.8e11 against 4.05e11.
  // particles per lane (line_ppt): one, or two whose maps interleave
  const int32_t ppt = line_ppt(style);
  std::vector<uint32_t> sigs;  // distinct element signatures of the line
  const std::string tables = deferred || flagged ? replay_tables(d, &sigs) : std::string();
  // a kernel with radiation steps and branches calls its RF sine out of line
  bool far_rf = false;
  if (rad_form != 0 && !flagged)
    for (const auto& k : d.kinds)
      for (uint32_t e : k) far_rf |= ((e & 0xffu) == K_MULT_CURV || (e & 0xffu) == K_MULT_LR);
  // the radiation step after a radiating multipole (rad_form): none or the
  // mode's; RADF, in a straight cell, with its tests collected
  std::string rad_macro;
  if (rad_form == 0)
    rad_macro = "#define RAD(kx, ky, lr, j) ((void)0)\n"
                "#define RADF(kx, ky, lr, ilr, j) ((void)0)\n";
  else
    rad_macro = std::string("#define RAD(kx, ky, lr, j) xtmm::radiate_at<") +
                (rad_form == 3 ? "true" : "false") + ">(q, kx, ky, lr, " +
                std::to_string(rad_form) +
                ", r.seed, pid, \\\n"
                "    t0 + t, ec + (j), r.gamma0, r.c_mean, r.c_quant, r.p0c, beta0, two_over_beta0, "
                "\\\n"
                "    r.photon_table, r.c_nphot, r.c_ucrit)\n"
                "#define RADF(kx, ky, lr, ilr, j) xtmm::radiate_flag<" +
                std::to_string(rad_form) + ">(q, kx, ky, lr, ilr, rr, ip0c, \\\n    " +
                (rad_form == 2 ? "xtmm::gauss_at(r.seed, pid, t0 + t, ec + (j), 0)" : "0.0") +
                ", beta0, two_over_beta0, bad)\n";
  const int32_t per_thread = (maxw + lanes - 1) / lanes;
  std::ostringstream s;
  s << "#include \"xtm_maps.h\"\n"
       "struct SoA { double *x, *px, *y, *py, *zeta, *delta, *ptau, *rpp, *rvv;\n"
       "             int *state, *at_element, *at_turn; long long* pid; };\n"
       "struct KRef { double beta0, two_over_beta0, gamma0, c_mean, c_quant, p0c;\n"
       "              unsigned long long seed; int rad_mode; int pad;\n"
       "              float* rec; int rec_turns; int rec_n;\n"
       "              const double* photon_table; double c_nphot, c_ucrit; };\n"
    << rad_macro <<
       "// a lane that fails a loss test stores the coordinates it entered the\n"
       "// element with (a rare, divergent store); the loss record follows at the end\n"
       "// (its slot index passes through a register move, so the nine store\n"
       "// addresses are formed on this rare path instead of held in registers)\n"
       "#define SAVE() do { int pj_ = pi; asm volatile(\"\" : \"+v\"(pj_)); \\\n"
       "    P.x[pj_] = q.x; P.px[pj_] = q.px; P.y[pj_] = q.y; P.py[pj_] = q.py; \\\n"
       "    P.zeta[pj_] = q.zeta; P.delta[pj_] = q.delta; P.ptau[pj_] = q.ptau; \\\n"
       "    P.rpp[pj_] = q.rpp; P.rvv[pj_] = q.rvv; } while (0)\n"
       "typedef const __attribute__((address_space(3))) double* lds_double;\n"
       "typedef const __attribute__((address_space(4))) double* cst_double;\n"
       "#define MAXW " << maxw << "\n"
       "#define PER_THREAD " << per_thread << "\n"
       "#define LANES " << lanes << "\n"
       "#define PPT " << ppt << "\n"
       << tables <<
       "extern \"C\" __global__ void __launch_bounds__(" << lanes << ")"
    << (scalar ? " __attribute__((amdgpu_waves_per_eu(3, 4)))\n" : "\n") <<
       "xtm_line(const double* __restrict__ " << (batched ? "prm_all" : "prm")
    << ", const int* __restrict__ cells, int n_cells,\n"
       "         int n_el, SoA P, const int* __restrict__ idx, const int* __restrict__ ctrl,\n"
       "         int n_turns, int backward, int n_min, int n_max, KRef r"
    << (batched ? ",\n         const int* __restrict__ first_slot, int nv, long long prm_stride"
                : "")
    << ") {\n";
  if (!scalar) s << "  __shared__ double slot[2 * MAXW];\n";
  s << "  const int lane = threadIdx.x;\n"
       "  (void)lane;\n"
       "  // another form serves this number of particles\n"
       "  if (ctrl[0] <= n_min || ctrl[0] > n_max) return;\n";
  // a batch of lattice variants with one cell structure: each slot belongs
  // to the variant whose slot range holds it; the wave makes one pass per
  // variant among its lanes (smallest first), reading that variant's
  // parameters, with the lanes of the other variants idle
  const std::string exit_stmt = batched ? "break;" : "return;";
  if (ppt == 1) {
    s << "  const int t0 = ctrl[1];\n"
         "  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;\n"
         "  const bool in_range = i < ctrl[0];\n"
         "  const int pi = in_range ? idx[i] : 0;\n";
    if (batched)
      s << "  const bool tracked0 = in_range && P.state[pi] == 1;\n"
           "  int v = 0x7fffffff;\n"
           "  if (tracked0) {\n"
           "    int lo = 0, hi = nv;\n"
           "    while (hi - lo > 1) { const int mid = (lo + hi) >> 1; "
           "if (first_slot[mid] <= pi) lo = mid; else hi = mid; }\n"
           "    v = lo;\n"
           "  }\n"
           "  bool pending = tracked0;\n"
           "  while (__any(pending)) {\n"
           "  int m_ = pending ? v : 0x7fffffff;\n"
           "  for (int o_ = 32; o_ > 0; o_ >>= 1) m_ = min(m_, __shfl_xor(m_, o_, 64));\n"
           "  const int vu = __builtin_amdgcn_readfirstlane(m_);\n"
           "  const bool tracked = pending && v == vu;\n"
           "  pending = pending && !tracked;\n"
           "  const double* __restrict__ prm = prm_all + (long long)vu * prm_stride;\n"
           "  do {\n";
    else
      s << "  const bool tracked = in_range && P.state[pi] == 1;\n";
    s << "  int code = tracked ? 0 : 1;\n"
         "  int st = 1;\n"
         "  bool live = tracked;\n";
    s << "  if (__syncthreads_and(code != 0)) " << exit_stmt << "\n";
    s << "  xtmm::Pt q;\n"
         "  q.x = P.x[pi]; q.px = P.px[pi]; q.y = P.y[pi]; q.py = P.py[pi]; q.zeta = P.zeta[pi];\n"
         "  q.delta = P.delta[pi]; q.ptau = P.ptau[pi]; q.rpp = P.rpp[pi]; q.rvv = P.rvv[pi];\n"
         "  const double beta0 = r.beta0, two_over_beta0 = r.two_over_beta0;\n"
         "  const long long pid = P.pid[pi];\n"
         "  xtmm::refresh(q, beta0);\n";
    if (flagged)
      s << "  double a_min = " << a_min_init(axis) << ";\n";
    if (flagged && rad_form != 0)
      s << "  // what the short radiation steps take for granted of their operands\n"
           "  // (in vector registers: the scalar ones are taken by the series' coefficients)\n"
           "  const xtmm::Rad rr{xtmm::in_vector(r.gamma0), xtmm::in_vector(r.c_mean),\n"
           "                     xtmm::in_vector(r.c_quant), xtmm::in_vector(r.p0c)};\n"
           "  const double ip0c = 1.0 / rr.p0c;\n"
           "  const bool rad_ok = (q.rpp == 1.0 / (1.0 + q.delta)) & (r.p0c >= 0x1p-100) &\n"
           "                      (r.p0c <= 0x1p100);\n";
  } else {
    // two particles per lane: slots i0 and i0 + LANES of the workgroup's range
    s << "  const int t0 = ctrl[1];\n"
         "  const long long i0 = (long long)blockIdx.x * (PPT * LANES) + threadIdx.x;\n"
         "  bool in_range_[PPT];\n"
         "  int pi_[PPT];\n"
         "#pragma unroll\n"
         "  for (int k_ = 0; k_ < PPT; ++k_) {\n"
         "    in_range_[k_] = i0 + k_ * LANES < ctrl[0];\n"
         "    pi_[k_] = in_range_[k_] ? idx[i0 + k_ * LANES] : 0;\n"
         "  }\n"
         "  bool tracked_[PPT];\n";
    if (batched)
      s << "  int v_[PPT];\n"
           "  bool pending_[PPT];\n"
           "#pragma unroll\n"
           "  for (int k_ = 0; k_ < PPT; ++k_) {\n"
           "    const int pi = pi_[k_];\n"
           "    pending_[k_] = in_range_[k_] && P.state[pi] == 1;\n"
           "    v_[k_] = 0x7fffffff;\n"
           "    if (pending_[k_]) {\n"
           "      int lo = 0, hi = nv;\n"
           "      while (hi - lo > 1) { const int mid = (lo + hi) >> 1; "
           "if (first_slot[mid] <= pi) lo = mid; else hi = mid; }\n"
           "      v_[k_] = lo;\n"
           "    }\n"
           "  }\n"
           "  while (__any(pending_[0] || pending_[1])) {\n"
           "  int m_ = min(pending_[0] ? v_[0] : 0x7fffffff, pending_[1] ? v_[1] : 0x7fffffff);\n"
           "  for (int o_ = 32; o_ > 0; o_ >>= 1) m_ = min(m_, __shfl_xor(m_, o_, 64));\n"
           "  const int vu = __builtin_amdgcn_readfirstlane(m_);\n"
           "#pragma unroll\n"
           "  for (int k_ = 0; k_ < PPT; ++k_) {\n"
           "    tracked_[k_] = pending_[k_] && v_[k_] == vu;\n"
           "    pending_[k_] = pending_[k_] && !tracked_[k_];\n"
           "  }\n"
           "  const double* __restrict__ prm = prm_all + (long long)vu * prm_stride;\n"
           "  do {\n";
    else
      s << "#pragma unroll\n"
           "  for (int k_ = 0; k_ < PPT; ++k_) tracked_[k_] = in_range_[k_] && P.state[pi_[k_]] == 1;\n";
    s << "  int code_[PPT], st_[PPT];\n"
         "  bool live_[PPT];\n"
         "#pragma unroll\n"
         "  for (int k_ = 0; k_ < PPT; ++k_) {\n"
         "    code_[k_] = tracked_[k_] ? 0 : 1; st_[k_] = 1; live_[k_] = tracked_[k_];\n"
         "  }\n"
         "  if (__syncthreads_and(code_[0] != 0 && code_[1] != 0)) " << exit_stmt << "\n"
         "  const double beta0 = r.beta0, two_over_beta0 = r.two_over_beta0;\n"
         "  xtmm::Pt q_[PPT];\n"
         "  long long pid_[PPT];\n"
         "#pragma unroll\n"
         "  for (int k_ = 0; k_ < PPT; ++k_) {\n"
         "    xtmm::Pt& q = q_[k_];\n"
         "    const int pi = pi_[k_];\n"
         "    q.x = P.x[pi]; q.px = P.px[pi]; q.y = P.y[pi]; q.py = P.py[pi]; q.zeta = P.zeta[pi];\n"
         "    q.delta = P.delta[pi]; q.ptau = P.ptau[pi]; q.rpp = P.rpp[pi]; q.rvv = P.rvv[pi];\n"
         "    pid_[k_] = P.pid[pi];\n"
         "    xtmm::refresh(q, beta0);\n"
         "  }\n";
  }
  if (!scalar)
    s << "  {\n"
         "    const int off0 = cells[1], nw0 = cells[3];\n"
         "    for (int w = lane; w < nw0; w += LANES) slot[w] = prm[off0 + w];\n"
         "  }\n"
         "  __syncthreads();\n"
         "  int b = 0;\n";
  // the cell table read one record (kind, first word, first element, words)
  // at a time, one cell ahead: the current cell's record came with the
  // previous cell's, so a cell starts with one scalar load, not three in
  // sequence
  s << "  const int4* __restrict__ cells4 = reinterpret_cast<const int4*>(cells);\n"
       "  int4 rc = cells4[0];\n"
       "  for (int t = 0; t < n_turns; ++t) {\n"
       "    const int enc_t = t * n_el + 1;\n";
  const std::string rec_body =
       "    if (r.rec && t0 + t < r.rec_turns && code == 0) {\n"
       "      const unsigned long long base = (unsigned long long)(t0 + t) * 4 * r.rec_n + pi;\n"
       "      r.rec[base] = (float)q.x;\n"
       "      r.rec[base + r.rec_n] = (float)q.px;\n"
       "      r.rec[base + 2ull * r.rec_n] = (float)q.y;\n"
       "      r.rec[base + 3ull * r.rec_n] = (float)q.py;\n"
       "    }\n";
  if (ppt == 1)
    s << rec_body;
  else
    s << "#pragma unroll\n"
         "    for (int k_ = 0; k_ < PPT; ++k_) {\n"
         "    const xtmm::Pt& q = q_[k_];\n"
         "    const int pi = pi_[k_], code = code_[k_];\n"
      << rec_body << "    }\n";
  s <<
       "    for (int c = 0; c < n_cells; ++c) {\n"
       "      const int cn = (c + 1 == n_cells) ? 0 : c + 1;\n"
       "      const int4 rn = cells4[cn];\n"
       "      const int kind = rc.x;\n"
       "      const int ec = rc.z;\n";
  if (!scalar)
    s << "      const int offn = rn.y, nwn = rn.w;\n"
         "      // every lane loads (past the cell's words, its first word; the\n"
         "      // parameter array ends in a pad word): no branch around the loads\n"
         "      double pre[PER_THREAD];\n"
         "#pragma unroll\n"
         "      for (int k = 0; k < PER_THREAD; ++k) {\n"
         "        const int w = lane + k * LANES;\n"
         "        const double v_ = prm[offn + (w < nwn ? w : 0)];\n"
         "        pre[k] = (w < nwn) ? v_ : 0.0;\n"
         "      }\n"
         "      // the slot as an LDS pointer passed through an empty register\n"
         "      // constraint: element reads become base + immediate-offset LDS loads\n"
         "      // instead of hoisted constant selects\n"
         "      lds_double p = (lds_double)slot + b * MAXW;\n"
         "      asm volatile(\"\" : \"+v\"(p));\n";
  else
    s << "      // the cell's words, read with scalar loads\n"
         "      cst_double p = (cst_double)(unsigned long long)(prm + rc.y);\n"
         "      asm volatile(\"\" : \"+s\"(p));\n";
  s <<
       "      // the cell's loss-code base lives in a VGPR so the per-element codes\n"
       "      // e0 + j are vector adds of literals, not hoisted scalar constants\n"
       "      int e0 = enc_t + ec;\n"
       "      asm volatile(\"\" : \"+v\"(e0));\n";
  if (deferred)
    s << "      const int code_in = code;\n"
         "      const xtmm::Pt qc = q;\n";
  if (flagged)
    s << "      const xtmm::Pt qc = q;\n"
         "      bool bad = !xtmm::drift_range(q)"
      << (rad_form != 0 ? " | !rad_ok" : "") << ";\n";
  for (size_t k = 0; k < d.kinds.size(); ++k) {
    s << "      " << (k ? "else if" : "if") << " (kind == " << k << ") {\n";
    const auto& kd = d.kinds[k];
    if (flagged) {
      straight_cell(s, kd, scalar, batched,
                    [](size_t) { return std::make_pair(std::string(), false); });
      s << "      }\n";
      continue;
    }
    std::vector<int32_t> off(kd.size() + 1, 0);
    for (size_t j = 0; j < kd.size(); ++j) off[j + 1] = off[j] + n_words(kd[j]);
    auto load = [&](size_t j) { read_words(s, kd[j], j, off[j]); };
    const std::vector<size_t> read_before = reads_ahead(kd);
    if (fetch == 2 && !kd.empty()) load(0);
    for (size_t j = 0; j < kd.size(); ++j) {
      std::string arr = "p + " + std::to_string(off[j]);
      if (fetch == 1) {
        load(j);
        s << "        __builtin_amdgcn_sched_barrier(0);\n";
      } else if (fetch == 2) {
        // fetch 2: the words of the elements to read ahead of this one
        for (size_t m = j + 1; m < kd.size() && m <= j + 2; ++m)
          if (read_before[m] == j) load(m);
        s << "        __builtin_amdgcn_sched_barrier(0);\n";
      }
      if (fetch != 0 && n_words(kd[j]) > 0) arr = "w" + std::to_string(j);
      const std::string stmt =
          emit(kd[j], arr, std::to_string(j), far_rf,
               deferred ? kMarkOnly : kSaveAtLoss);
      if (stmt.empty()) continue;
      if (ppt == 1) {
        s << "        " << stmt << "\n";
      } else {
        // the same element for each particle of the lane, through references
        // that give each copy the one-particle names
        for (int32_t k = 0; k < ppt; ++k)
          s << "        { xtmm::Pt& q = q_[" << k << "]; int& code = code_[" << k
            << "]; int& st = st_[" << k << "]; bool& live = live_[" << k
            << "]; (void)live; const int pi = pi_[" << k
            << "]; const long long pid = pid_[" << k << "]; (void)pid; (void)pi; " << stmt
            << " }\n";
      }
    }
    s << "      }\n";
  }
  if (deferred) {
    // one wave-uniform test per cell; a lane lost in the cell re-applies the
    // cell's maps up to its lost element from the cell-entry copy (the same
    // operations, so the same values) and stores those entry coordinates.
    // The replay walks the cell's element list with one switch over the
    // line's element signatures, so this rare path adds little code.
    s << "      if (__any(code != code_in)) {\n"
         "        if (code != code_in) {\n"
         "          const int jl = code - e0;\n"
         "          xtmm::Pt q = qc;\n"
         "          for (int j = kind_first[kind]; j < kind_first[kind] + jl; ++j) {\n"
         "            const double* pe = p + elem_off[j];\n"
         "            switch (elem_sig[j]) {\n";
    for (size_t g = 0; g < sigs.size(); ++g) {
      const std::string stmt = emit(sigs[g], "pe", "(j - kind_first[kind])", far_rf, kReplay);
      if (!stmt.empty()) s << "              case " << g << ": " << stmt << " break;\n";
    }
    s << "              default: break;\n"
         "            }\n"
         "          }\n"
         "          SAVE();\n"
         "        }\n"
         "      }\n";
  }
  if (flagged) {
    // the rare second pass through the cell: from the entry copy, element by
    // element, with the generic drift and the loss test where they belong
    s << "      bad |= !(q.x == q.x);\n"
         "      bad &= live;\n"
         "      if (__builtin_expect(__builtin_amdgcn_ballot_w64(bad) != 0, 0)) {\n"
         "        if (bad) {\n"
         "          q = qc;\n"
      << (scalar ? "          const int4 rr = cells4[c];\n          const int kind = rr.x;\n" : "") <<
         "          for (int j = kind_first[kind]; j < kind_first[kind + 1]; ++j) {\n"
      << (scalar ? "            const double* pe = prm + rr.y + elem_off[j];\n"
                 : "            const double* pe = (const double*)(p + elem_off[j]);\n")
      << "            const xtmm::Pt q0 = q;\n"
         "            bool ok = true;\n"
         "            int ls = 0;\n"
         "            switch (elem_sig[j]) {\n";
    for (size_t g = 0; g < sigs.size(); ++g) {
      const std::string stmt = emit(sigs[g], "pe", "(j - kind_first[kind])", far_rf,
                                    scalar ? kTestScalar : kTest, batched, scalar);
      if (!stmt.empty()) s << "              case " << g << ": " << stmt << " break;\n";
    }
    s << "              default: break;\n"
         "            }\n"
         "            if (!ok && live) {\n"
         "              const xtmm::Pt q = q0;\n"
         "              SAVE(); code = e0 + (j - kind_first[kind]); st = ls; live = false;\n"
         "            }\n"
         "          }\n"
         "        }\n"
         "      }\n";
  }
  if (!scalar)
  s << "#pragma unroll\n"
       "      for (int k = 0; k < PER_THREAD; ++k) {\n"
       "        const int w = lane + k * LANES;\n"
       "        if (w < nwn) slot[(b ^ 1) * MAXW + w] = pre[k];\n"
       "      }\n"
       "      b ^= 1;\n";
  s << "      rc = rn;\n";
  if (!scalar) s << "      __syncthreads();\n";
  s << "    }\n";
  if (ppt == 1)
    s << "    if (__syncthreads_and(code != 0)) break;\n";
  else
    s << "    if (__syncthreads_and(code_[0] != 0 && code_[1] != 0)) break;\n";
  const std::string store_body =
       "  if (code == 0) {\n"
       "    P.x[pi] = q.x; P.px[pi] = q.px; P.y[pi] = q.y; P.py[pi] = q.py; P.zeta[pi] = q.zeta;\n"
       "    P.delta[pi] = q.delta; P.ptau[pi] = q.ptau; P.rpp[pi] = q.rpp; P.rvv[pi] = q.rvv;\n"
       "    P.at_turn[pi] = backward ? t0 - n_turns : t0 + n_turns;\n"
       "    P.at_element[pi] = 0;\n"
       "  } else {\n"
       "    const int tl = (code - 1) / n_el, el = (code - 1) - tl * n_el;\n"
       "    P.state[pi] = st;\n"
       "    P.at_element[pi] = backward ? n_el - 1 - el : el;\n"
       "    P.at_turn[pi] = backward ? t0 - 1 - tl : t0 + tl;\n"
       "  }\n";
  s << "  }\n";
  if (ppt == 1)
    s << "  if (!tracked) " << exit_stmt << "\n" << store_body;
  else
    s << "#pragma unroll\n"
         "  for (int k_ = 0; k_ < PPT; ++k_) {\n"
         "  if (!tracked_[k_]) continue;\n"
         "  const xtmm::Pt& q = q_[k_];\n"
         "  const int pi = pi_[k_], code = code_[k_], st = st_[k_];\n"
      << store_body << "  }\n";
  if (batched)
    s << "  } while (0);\n"
         "  }\n";
  s << "}\n";
  return s.str();
}

// Generated recording kernel for optics by tracking: one turn of a few
// particles from their (x, px, y, py, zeta, delta), the coordinates stored at
// the entry of every element and after the last.  Apertures are not applied,
// and a lane whose drift finds no real longitudinal momentum keeps its entry
// coordinates and applies no further maps.
//   What bounds it: one wave's chain of dependent operations through the line.
// So the wave that tracks does nothing else: cells are straight as in the
// tracking kernel (see generate), a lane that failed a test going through its
// cell again, rows leave as each element is entered, and the cell's parameters
// are brought to LDS by a second wave, kAhead cells ahead (a lone lattice's
// words come from beyond the L2).  Optics of the 20,000-element DA ring, a
// probe turn of 11 particles with every row: 2.4 ms; 5.1 ms when the tracking
// wave also staged parameters and moved each cell's rows through LDS, with a
// branch per drift.
std::string generate_record(const Decomp& d, bool axis) {
  int32_t maxw = 1;
  for (const auto& k : d.kinds) maxw = std::max(maxw, kind_words(k));
  constexpr int32_t lanes = 64;
  const int32_t per_thread = (maxw + lanes - 1) / lanes;
  std::vector<uint32_t> sigs;
  const std::string tables = replay_tables(d, &sigs);
  std::ostringstream s;
  s << "#include \"xtm_maps.h\"\n"
       "struct KRef { double beta0, two_over_beta0, gamma0, c_mean, c_quant, p0c;\n"
       "              unsigned long long seed; int rad_mode; int pad;\n"
       "              float* rec; int rec_turns; int rec_n;\n"
       "              const double* photon_table; double c_nphot, c_ucrit; };\n"
       "#define RAD(kx, ky, lr, j) ((void)0)\n"
       "#define RADF(kx, ky, lr, ilr, j) ((void)0)\n"
       "typedef const __attribute__((address_space(3))) double* lds_double;\n"
       "#define MAXW " << maxw << "\n"
       "#define PER_THREAD " << per_thread << "\n"
       "#define LANES " << lanes << "\n"
       "#define AHEAD " << kAhead << "\n"
    << tables <<
       "// the lane's row of the element entered, and on to the next element's\n"
       "#define ROW(to) do { (to)[0] = make_double2(q.x, q.px); \\\n"
       "    (to)[1] = make_double2(q.y, q.py); (to)[2] = make_double2(q.zeta, q.delta); \\\n"
       "    (to) += row; } while (0)\n"
       "// (LDS only: the rows on their way to memory are not waited for)\n"
       "// (no access moves across it: neither a store behind the wait that is for it\n"
       "// nor a read ahead of the barrier)\n"
       "#define BARRIER() do { asm volatile(\"\" ::: \"memory\"); \\\n"
       "    __builtin_amdgcn_s_waitcnt(0xc07f); __builtin_amdgcn_s_barrier(); \\\n"
       "    asm volatile(\"\" ::: \"memory\"); } while (0)\n"
       "extern \"C\" __global__ void __launch_bounds__(2 * LANES)\n"
       "// (prm without __restrict__: its loads then stay before the barriers they are\n"
       "// written before, instead of sinking to their use)\n"
       "xtm_record(const double* prm, const int* __restrict__ cells, int n_cells,\n"
       "           int n_el, const double* __restrict__ c6, long long n,\n"
       "           double* __restrict__ out, KRef r) {\n"
       "  __shared__ double slot[2 * MAXW];\n"
       "  const int lane = threadIdx.x & (LANES - 1);\n"
       "  // (constant address space: scalar loads on either side of the barriers)\n"
       "  typedef int cell __attribute__((ext_vector_type(4)));\n"
       "  const __attribute__((address_space(4))) cell* cells4 =\n"
       "      (const __attribute__((address_space(4))) cell*)(unsigned long long)cells;\n"
       "  if (__builtin_amdgcn_readfirstlane(threadIdx.x) >= LANES) {\n"
       "    // cell c's words lie in slot c % 2 from the barrier before it; set\n"
       "    // k % AHEAD of registers holds those of cell k on their way.  Every lane\n"
       "    // loads (past the cell's words its first, past the line its last cell; the\n"
       "    // parameter array ends in a pad word), so no load is under a branch.\n"
       "    double pre[AHEAD][PER_THREAD];\n"
       "    auto load = [&](int k, int c) {\n"
       "      const cell rc = cells4[c < n_cells ? c : n_cells - 1];\n"
       "#pragma unroll\n"
       "      for (int m = 0; m < PER_THREAD; ++m) {\n"
       "        const int w = lane + m * LANES;\n"
       "        pre[k][m] = prm[rc.y + (w < rc.w ? w : 0)];\n"
       "      }\n"
       "    };\n"
       "#pragma unroll\n"
       "    for (int k = 0; k < AHEAD; ++k) load(k, k);\n"
       "    for (int c = 0; c <= n_cells; c += AHEAD) {\n"
       "#pragma unroll\n"
       "      for (int k = 0; k < AHEAD; ++k) {\n"
       "        if (c + k > n_cells) break;\n"
       "        // cell c + k into its slot while the other wave tracks cell c + k - 1\n"
       "#pragma unroll\n"
       "        for (int m = 0; m < PER_THREAD; ++m) {\n"
       "          const int w = lane + m * LANES;\n"
       "          if (w < MAXW) slot[((c + k) & 1) * MAXW + w] = pre[k][m];\n"
       "        }\n"
       "        load(k, c + k + AHEAD);\n"
       "        BARRIER();\n"
       "      }\n"
       "    }\n"
       "    return;\n"
       "  }\n"
       "  const long long i = (long long)blockIdx.x * LANES + lane;\n"
       "  const bool act = i < n;\n"
       "  const double beta0 = r.beta0, two_over_beta0 = r.two_over_beta0;\n"
       "  (void)two_over_beta0;\n"
       "  xtmm::Pt q{};\n"
       "  if (act) {\n"
       "    const double* c = c6 + 6 * i;\n"
       "    const double dl = c[5];\n"
       "    const double u = dl * (2.0 + dl);\n"
       "    q.x = c[0]; q.px = c[1]; q.y = c[2]; q.py = c[3]; q.zeta = c[4]; q.delta = dl;\n"
       "    q.ptau = beta0 * u / (1.0 + sqrt(1.0 + beta0 * beta0 * u));\n"
       "    q.rpp = 1.0 / (1.0 + dl);\n"
       "    q.rvv = (1.0 + dl) / (1.0 + beta0 * q.ptau);\n"
       "    xtmm::refresh(q, beta0);\n"
       "  }\n"
       "  double a_min = " << a_min_init(axis) << ";\n"
       "  const unsigned long long row = 3ull * n;\n"
       "  double2* __restrict__ to = reinterpret_cast<double2*>(out) + 3 * i;\n"
       "  bool alive = act;\n"
       "  cell rc = cells4[0];\n"
       "  BARRIER();\n"
       "  for (int c = 0; c < n_cells; ++c) {\n"
       "    const cell rn = cells4[c + 1 < n_cells ? c + 1 : c];\n"
       "    const int kind = rc.x;\n"
       "    double2* from = to;\n"
       "    lds_double p = (lds_double)slot + (c & 1) * MAXW;\n"
       "    asm volatile(\"\" : \"+v\"(p));\n"
       "    const xtmm::Pt qc = q;\n"
       "    // a lane that keeps its coordinates takes the second pass alone\n"
       "    bool bad = !xtmm::drift_range(q) | !alive;\n"
       "    if (act) {\n";
  for (size_t k = 0; k < d.kinds.size(); ++k) {
    s << "    " << (k ? "else if" : "if") << " (kind == " << k << ") {\n";
    straight_cell(s, d.kinds[k], false, false, [&](size_t j) {
      const uint32_t kt = d.kinds[k][j] & 0xffu;
      return std::make_pair(std::string("ROW(to);"), kt == K_AP_CIRC || kt == K_AP_ELL || kt == K_AP_RECT);
    });
    s << "    }\n";
  }
  s << "    }\n"
       "    bad |= !(q.x == q.x);\n"
       "    bad &= act;\n"
       "    if (__builtin_expect(__builtin_amdgcn_ballot_w64(bad) != 0, 0)) {\n"
       "      if (bad) {\n"
       "        q = qc;\n"
       "        double2* ta = from;\n"
       "        for (int j = kind_first[kind]; j < kind_first[kind + 1]; ++j) {\n"
       "          const double* pe = (const double*)(p + elem_off[j]);\n"
       "          ROW(ta);\n"
       "          if (!alive) continue;\n"
       "          const xtmm::Pt q0 = q;\n"
       "          bool ok = true;\n"
       "          int ls = 0;\n"
       "          switch (elem_sig[j]) {\n";
  for (size_t g = 0; g < sigs.size(); ++g) {
    const uint32_t kt = sigs[g] & 0xffu;
    if (kt == K_AP_CIRC || kt == K_AP_ELL || kt == K_AP_RECT) continue;
    const std::string stmt = emit(sigs[g], "pe", "0", false, kTest);
    if (!stmt.empty()) s << "            case " << g << ": " << stmt << " break;\n";
  }
  s << "            default: break;\n"
       "          }\n"
       "          (void)ls;\n"
       "          if (!ok) { q = q0; alive = false; }\n"
       "        }\n"
       "      }\n"
       "    }\n"
       "    rc = rn;\n"
       "    BARRIER();\n"
       "  }\n"
       "  if (act) ROW(to);\n"
       "}\n";
  return s.str();
}

// ilp_sched: LLVM's instruction-level-parallelism scheduling strategy instead
// of the default occupancy-first one.  A particle's element chain is one
// dependent sequence and, in the tail of a dynamic-aperture scan, a wave is
// alone on its SIMD and waits on each result; the ILP schedule interleaves
// more of each element's independent operations at the cost of registers
// (the DA-ring kernel: 205 VGPRs against 175).
Compiled compile(const std::string& src, const char* name, bool ilp_sched) {
  Compiled out;
  hiprtcProgram prog;
  const char* hdr = kMapsSource;
  const char* hname = "xtm_maps.h";
  if (hiprtcCreateProgram(&prog, src.c_str(), "xtm_line.hip", 1, &hdr, &hname) != HIPRTC_SUCCESS) {
    out.error = "hiprtcCreateProgram failed";
    return out;
  }
  std::vector<const char*> opts = {"--offload-arch=gfx950", "-O3", "-std=c++17",
                                   "-ffp-contract=off", "-fno-fast-math", "-Xclang",
                                   "-target-feature", "-Xclang", "-packed-fp32-ops"};
  if (ilp_sched) {
    opts.push_back("-mllvm");
    opts.push_back("-amdgpu-sched-strategy=max-ilp");
  }
  hiprtcResult r = hiprtcCompileProgram(prog, (int)opts.size(), opts.data());
  if (r != HIPRTC_SUCCESS) {
    size_t ls = 0;
    hiprtcGetProgramLogSize(prog, &ls);
    std::string log(ls, '\0');
    if (ls) hiprtcGetProgramLog(prog, &log[0]);
    out.error = "hiprtc: " + log;
    hiprtcDestroyProgram(&prog);
    return out;
  }
  size_t cs = 0;
  hiprtcGetCodeSize(prog, &cs);
  std::vector<char> code(cs);
  hiprtcGetCode(prog, code.data());
  hiprtcDestroyProgram(&prog);
  if (hipModuleLoadData(&out.module, code.data()) != hipSuccess) {
    out.error = "hipModuleLoadData failed";
    return out;
  }
  if (hipModuleGetFunction(&out.fn, out.module, name) != hipSuccess) {
    out.error = "hipModuleGetFunction failed";
    out.fn = nullptr;
  }
  return out;
}

}  // namespace

namespace {
// Signature, parameter-word position and parameter words of each element of
// a host element table.  curv, rad: the parameters of a bend with a curvature
// term and of a multipole with a radiation length alone are followed by the
// reciprocal of that length, their last word.
void split_table(const std::vector<uint64_t>& tab, int32_t n_el, std::vector<uint32_t>* sig,
                 std::vector<int32_t>* word_of, std::vector<double>* prm, bool curv = false,
                 bool rad = false) {
  size_t off = 0;
  for (int32_t e = 0; e < n_el; ++e) {
    const uint64_t h = tab[off];
    const uint32_t nw = (uint32_t)((h >> 16) & 0xffffu);
    sig->push_back(sig_of(h));
    word_of->push_back((int32_t)prm->size());
    for (uint32_t w = 0; w < nw; ++w) {
      double d;
      std::memcpy(&d, &tab[off + 1 + w], 8);
      prm->push_back(d);
    }
    const uint32_t kt = (uint32_t)(h & 0xffu);
    if ((curv && kt == K_MULT_CURV) || (rad && kt == K_MULT_LR)) {
      sig->back() |= kRecip;
      prm->push_back(1.0 / prm->back());
    }
    off += 1 + nw;
  }
}

// The words of an element (n_words of them) as the wide form reads them: the
// addends of its multiply-adds negated (xtmm::addend), which are a drift's
// length and a multipole's coefficients below the highest order.
void wide_words(uint32_t sig, double* w) {
  const uint32_t kt = sig & 0xffu, order = (sig >> 8) & 0xffu;
  if (kt == K_DRIFT) w[0] = -w[0];
  if (kt == K_MULT || kt == K_MULT_CURV || kt == K_MULT_LR)
    for (uint32_t m = 2; m < 2 * (order + 1); ++m) w[m] = -w[m];
}

// Whether the short sequences of the curvature term serve every bend of a
// table (curv), and those of the radiation step every radiating element (rad).
void short_lengths(const std::vector<uint64_t>& tab, int32_t n_el, bool* curv, bool* rad) {
  auto in_range = [](uint64_t w) {
    double v;
    std::memcpy(&v, &w, 8);
    return std::fabs(v) >= 0x1p-100 && std::fabs(v) <= 0x1p100;
  };
  size_t off = 0;
  for (int32_t e = 0; e < n_el; ++e) {
    const uint32_t kt = (uint32_t)(tab[off] & 0xffu), nw = (uint32_t)((tab[off] >> 16) & 0xffffu);
    if (kt == K_MULT_CURV || kt == K_MULT_LR) {  // the length is the last word
      const bool ok = in_range(tab[off + nw]) && !(tab[off + nw] >> 63);
      *rad &= ok;
      if (kt == K_MULT_CURV) *curv &= ok && in_range(tab[off + nw - 2]);
    }
    off += 1 + nw;
  }
}
}  // namespace

// Whether a line without radiation keeps a particle on the axis with the
// reference momentum there until its momentum changes: no shift, no dipole kick
// but one that the curvature takes back (knl0 = hxl).
static bool keeps_axis(const std::vector<uint64_t>& tab, int32_t n_el) {
  auto word = [&](size_t at) {
    double v;
    std::memcpy(&v, &tab[at], 8);
    return v;
  };
  size_t off = 0;
  for (int32_t e = 0; e < n_el; ++e) {
    const uint32_t kt = (uint32_t)(tab[off] & 0xffu), order = (uint32_t)((tab[off] >> 8) & 0xffu);
    const size_t c0 = off + 1 + 2 * order;  // the dipole term's words
    if (kt == K_SHIFT && (word(off + 1) != 0.0 || word(off + 2) != 0.0)) return false;
    if (kt == K_MULT || kt == K_MULT_LR || kt == K_MULT_CURV) {
      const double back = kt == K_MULT_CURV ? word(c0 + 2) : 0.0;
      if (word(c0) != back || word(c0 + 1) != 0.0) return false;
    }
    off += 1 + (size_t)((tab[off] >> 16) & 0xffffu);
  }
  return true;
}

bool table_radiates(const std::vector<uint64_t>& tab, int32_t n_el) {
  size_t off = 0;
  for (int32_t e = 0; e < n_el && off < tab.size(); ++e) {
    const uint32_t kt = (uint32_t)(tab[off] & 0xffu);
    if (kt == K_MULT_CURV || kt == K_MULT_LR) return true;
    off += 1 + (size_t)((tab[off] >> 16) & 0xffffu);
  }
  return false;
}

bool build_line_kernel(const std::vector<uint64_t>& tab, int32_t n_el, int32_t style,
                       int32_t rad_form, LineKernel* k) {
  return build_line_kernel_multi({&tab}, n_el, style, false, rad_form, k);
}

namespace {
// Compile a generated kernel, or take it from the cache; null on failure.
hipFunction_t cached_function(const std::string& source, const char* name, bool ilp_sched,
                              std::string* error) {
  std::lock_guard<std::mutex> lock(g_mu);
  const std::string key = (ilp_sched ? "ilp\n" : "default\n") + source;
  auto it = g_cache.find(key);
  if (it == g_cache.end()) it = g_cache.emplace(key, compile(source, name, ilp_sched)).first;
  if (!it->second.fn) *error = it->second.error;
  return it->second.fn;
}

// Compile (or take from the cache) a generated kernel and upload its
// parameter array and cell table.
bool finish_kernel(const Decomp& d, const std::string& source, const char* name,
                   bool ilp_sched, const std::vector<int32_t>& word_of,
                   const std::vector<double>& prm, LineKernel* k) {
  k->source = source;
  k->fn = cached_function(source, name, ilp_sched, &k->error);
  if (!k->fn) return false;
  std::vector<int32_t> cells;  // per cell: kind, first parameter word, first element, words
  for (size_t c = 0; c < d.cell_kind.size(); ++c) {
    cells.push_back(d.cell_kind[c]);
    cells.push_back(word_of[d.cell_start[c]]);
    cells.push_back(d.cell_start[c]);
    cells.push_back(kind_words(d.kinds[d.cell_kind[c]]));
  }
  k->period = (int32_t)d.kinds[0].size();
  k->n_cells = (int32_t)d.cell_kind.size();
  k->n_kinds = (int32_t)d.kinds.size();
  if (hipMalloc(&k->prm_d, prm.size() * sizeof(double)) != hipSuccess ||
      hipMalloc(&k->cells_d, cells.size() * sizeof(int32_t)) != hipSuccess ||
      hipMemcpy(k->prm_d, prm.data(), prm.size() * sizeof(double), hipMemcpyHostToDevice) !=
          hipSuccess ||
      hipMemcpy(k->cells_d, cells.data(), cells.size() * sizeof(int32_t),
                hipMemcpyHostToDevice) != hipSuccess) {
    k->error = "device allocation for the line kernel failed";
    free_line_kernel(k);
    return false;
  }
  k->ok = true;
  return true;
}
}  // namespace

bool build_line_kernel_multi(const std::vector<const std::vector<uint64_t>*>& tabs, int32_t n_el,
                             int32_t style, bool batched, int32_t rad_form, LineKernel* k) {
  std::vector<uint32_t> sig;
  std::vector<int32_t> word_of;  // parameter-array offset of each element
  std::vector<double> prm;
  sig.reserve(n_el);
  bool curv = line_long(style), rad = rad_form != 0;
  for (const auto* t : tabs) short_lengths(*t, n_el, &curv, &rad);
  // straight cells: no photon emitter (its loop is a branch), and the mean and
  // Gaussian models where every radiation length suits their short sequences
  const bool flagged = line_long(style) && (rad_form == 0 || (rad_form != 3 && curv && rad));
  curv &= flagged;
  rad &= flagged;
  bool axis = flagged && rad_form == 0;
  for (size_t v = 0; v < tabs.size() && axis; ++v) axis = keeps_axis(*tabs[v], n_el);
  split_table(*tabs[0], n_el, &sig, &word_of, &prm, curv, rad);
  if (prm.empty()) prm.push_back(0.0);
  const size_t stride = prm.size();
  for (size_t v = 1; v < tabs.size(); ++v) {
    std::vector<uint32_t> sv;
    std::vector<int32_t> wv;
    std::vector<double> pv;
    split_table(*tabs[v], n_el, &sv, &wv, &pv, curv, rad);
    if (pv.empty()) pv.push_back(0.0);
    if (sv != sig || pv.size() != stride) {
      k->error = "lattice variant " + std::to_string(v) + " differs in element structure";
      return false;
    }
    prm.insert(prm.end(), pv.begin(), pv.end());
  }
  prm.push_back(0.0);  // pad word: the first word of a cell without words
  if (batched && line_block(style) != 64) {
    k->error = "batched per-line kernels use one-wave workgroups";
    return false;
  }
  Decomp d;
  if (!decompose(sig, &d, line_long(style) ? kLongUnit : kMaxUnit,
                 line_long(style) ? kLongCode : kMaxCode)) {
    k->error = "no cell decomposition within the code budget";
    return false;
  }
  k->style = style;
  k->batched = batched;
  k->nv = (int32_t)tabs.size();
  k->stride = (int64_t)stride;
  // single-lattice kernels take the ILP schedule (measured 2-4 % faster on
  // the DA ring and with the mean and Gaussian radiation, 1 % slower on a
  // saturated FODO ring); the batched ones (0.7 % slower with it on 64
  // variants) and the photon form (4 % slower) keep the default; the straight
  // cells take it (with the default, 200 registers instead of 141 on the FODO
  // ring and 9.4 ms instead of 8.8 ms for 1M particles)
  const bool ilp = flagged || (!batched && rad_form != 3);
  // (no wide form with radiation, whose constants need the scalar registers:
  // electron ring, 131,072 particles, two turns, 13.3 ms against 11.3 ms)
  const bool wide = flagged && rad_form == 0;
  if (wide) k->wide_source = generate(d, style, batched, 0, true, true, axis);
  if (!finish_kernel(d, generate(d, style, batched, rad_form, flagged, false, axis), "xtm_line", ilp,
                     word_of, prm, k))
    return false;
  if (wide) {
    k->wide_prm = std::move(prm);
    k->wide_sig = std::move(sig);
    k->wide_word = std::move(word_of);
  }
  return true;
}

bool is_capturing(hipStream_t s) {
  hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(s, &c) == hipSuccess && c != hipStreamCaptureStatusNone;
}

void build_wide_form(LineKernel* k, hipStream_t s) {
  if (!k->ok || k->wide_tried || k->wide_source.empty() || is_capturing(s)) return;
  k->wide_tried = true;
  std::vector<double> prm = std::move(k->wide_prm);
  const std::vector<uint32_t> sig = std::move(k->wide_sig);
  const std::vector<int32_t> word_of = std::move(k->wide_word);
  const hipFunction_t fn = cached_function(k->wide_source, "xtm_line", true, &k->wide_error);
  if (!fn) return;
  for (int32_t v = 0; v < k->nv; ++v)
    for (size_t e = 0; e < sig.size(); ++e) wide_words(sig[e], &prm[v * k->stride + word_of[e]]);
  const size_t bytes = prm.size() * sizeof(double);
  if (hipMalloc(&k->wide_prm_d, bytes) != hipSuccess ||
      hipMemcpy(k->wide_prm_d, prm.data(), bytes, hipMemcpyHostToDevice) != hipSuccess) {
    hipFree(k->wide_prm_d);
    k->wide_prm_d = nullptr;
    k->wide_error = "device allocation for the wide form failed";
    return;
  }
  k->wide_fn = fn;
}

bool build_record_kernel(const std::vector<uint64_t>& tab, int32_t n_el, LineKernel* k) {
  std::vector<uint32_t> sig;
  std::vector<int32_t> word_of;
  std::vector<double> prm;
  bool curv = true, rad = false;
  short_lengths(tab, n_el, &curv, &rad);
  split_table(tab, n_el, &sig, &word_of, &prm, curv);
  prm.push_back(0.0);  // pad word: the first word of a cell without words
  Decomp d;
  if (!decompose(sig, &d, kLongUnit, kLongCode)) {
    k->error = "no cell decomposition within the code budget";
    return false;
  }
  k->style = 5;
  k->stride = (int64_t)prm.size();
  return finish_kernel(d, generate_record(d, keeps_axis(tab, n_el)), "xtm_record", true, word_of, prm, k);
}

void free_line_kernel(LineKernel* k) {
  hipFree(k->prm_d);
  hipFree(k->cells_d);
  hipFree(k->wide_prm_d);
  k->prm_d = nullptr;
  k->wide_prm_d = nullptr;
  k->wide_fn = nullptr;
  k->cells_d = nullptr;
  k->ok = false;
}

// The launches of one chunk.  A set that may hold more particles than one wave
// per SIMD (kWideParticles) is launched on the wide form, which reads its
// parameters with scalar loads, and on the form that stages them in LDS: the
// alive count is on the device, and each launch ends at once unless the count
// is its own.  `args` holds the kernel arguments, the parameters at `prm` and
// the bounds at `n_min` and `n_max`.
namespace {
hipError_t launch_forms(const LineKernel& k, int64_t grid_upper, void** args, const double** prm,
                        int32_t* n_min, int32_t* n_max, hipStream_t s) {
  const int32_t wg = line_block(k.style);
  const int64_t per_wg = (int64_t)wg * line_ppt(k.style);  // particles per workgroup
  const bool wide = k.wide_fn && grid_upper > kWideParticles;
  *prm = k.prm_d;
  *n_min = -1;
  *n_max = wide ? kWideParticles : INT32_MAX;
  const int64_t upper = wide ? kWideParticles : grid_upper;
  hipError_t e = hipModuleLaunchKernel(k.fn, (unsigned)((upper + per_wg - 1) / per_wg), 1, 1,
                                       (unsigned)wg, 1, 1, 0, s, args, nullptr);
  if (e != hipSuccess || !wide) return e;
  *prm = k.wide_prm_d;
  *n_min = kWideParticles;
  *n_max = INT32_MAX;
  ++k.wide_launches;
  return hipModuleLaunchKernel(k.wide_fn, (unsigned)((grid_upper + per_wg - 1) / per_wg), 1, 1,
                               (unsigned)wg, 1, 1, 0, s, args, nullptr);
}
}  // namespace

hipError_t launch_line(const LineKernel& k, int32_t n_el, SoA P, const int32_t* idx,
                       const int32_t* ctrl, int64_t grid_upper, int32_t n_turns,
                       int32_t backward, KernelRef r, hipStream_t s) {
  if (grid_upper <= 0 || n_turns <= 0) return hipSuccess;
  const double* prm = nullptr;
  const int32_t* cells = k.cells_d;
  int32_t n_cells = k.n_cells, n_min = 0, n_max = 0;
  void* args[] = {(void*)&prm, (void*)&cells, (void*)&n_cells, (void*)&n_el, (void*)&P,
                  (void*)&idx, (void*)&ctrl, (void*)&n_turns, (void*)&backward, (void*)&n_min,
                  (void*)&n_max, (void*)&r};
  return launch_forms(k, grid_upper, args, &prm, &n_min, &n_max, s);
}

hipError_t launch_line_record(const LineKernel& k, int32_t n_el, const double* c6, int64_t n,
                              double* out, KernelRef r, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const double* prm = k.prm_d;
  const int32_t* cells = k.cells_d;
  int32_t n_cells = k.n_cells;
  long long nn = (long long)n;
  void* args[] = {(void*)&prm, (void*)&cells, (void*)&n_cells, (void*)&n_el, (void*)&c6,
                  (void*)&nn,  (void*)&out,   (void*)&r};
  const unsigned grid = (unsigned)((n + 63) / 64);
  return hipModuleLaunchKernel(k.fn, grid, 1, 1, 128, 1, 1, 0, s, args, nullptr);
}

hipError_t launch_line_batched(const LineKernel& k, int32_t n_el, SoA P, const int32_t* idx,
                               const int32_t* ctrl, int64_t grid_upper, int32_t n_turns,
                               int32_t backward, KernelRef r, const int32_t* first_slot,
                               hipStream_t s) {
  if (grid_upper <= 0 || n_turns <= 0) return hipSuccess;
  if (!k.batched) return hipErrorInvalidValue;
  const double* prm = nullptr;
  const int32_t* cells = k.cells_d;
  int32_t n_cells = k.n_cells, nv = k.nv, n_min = 0, n_max = 0;
  long long stride = (long long)k.stride;
  void* args[] = {(void*)&prm,  (void*)&cells, (void*)&n_cells, (void*)&n_el,
                  (void*)&P,    (void*)&idx,   (void*)&ctrl,    (void*)&n_turns,
                  (void*)&backward, (void*)&n_min, (void*)&n_max, (void*)&r,
                  (void*)&first_slot, (void*)&nv, (void*)&stride};
  return launch_forms(k, grid_upper, args, &prm, &n_min, &n_max, s);
}

}  // namespace xtm
