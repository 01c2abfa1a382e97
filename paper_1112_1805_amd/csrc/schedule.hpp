// Launch schedules of the mixed-radix path: the stage lists a transform can run, the shapes a row
// pass can be launched with, and the lines of a schedule cache file.  Plain C++ (no device code).
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

namespace shs {

constexpr int kMaxStages = 10;
constexpr int kFirstRadix = 32;   // extra radix of a column transform's first stage
struct FftPlan {
  int L;                     // transform length
  int ns;                    // number of stages
  int radix[kMaxStages];     // product = L
  // Division by the stage stride Ns_s = radix[0] * ... * radix[s-1] without a divide:
  // x / Ns_s = (umulhi(x, mag[s]) + x) >> sh[s] for x < 2^21 (constants from the host).
  unsigned mag[kMaxStages];
  int sh[kMaxStages];
};
// LDS buffers of one strip a column transform needs between its stages.
inline int col_bufs(const FftPlan& pl) { return pl.ns > 2 ? 2 : 1; }

// The radices a stage can have; with_radix calls f with the radix as a compile-time value.
#define SHS_RADICES(X)                                                                     \
  X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17)  \
  X(18) X(19) X(20) X(22) X(23) X(24)

// Entries of the twiddle tables that row and column passes copy into LDS (contents: generic.hpp).
constexpr int row_tab_len(int n) { return 3 * (n / 2); }
constexpr int col_tab_len(int n) { return n; }

constexpr int kGenericMaxN = 1024;          // largest image side of the mixed-radix path
constexpr size_t kRowGLdsMax = 64 * 1024;   // dynamic LDS a generic row block may take

// LDS buffers a row-pass wave needs for rw rows: one where every stage is a single pass over
// the wave's 64 lanes (all its reads precede its writes), else two.
inline int row_g_bufs(const FftPlan& pl, int rw) {
  int rmin = pl.radix[0];
  for (int i = 1; i < pl.ns; ++i) rmin = pl.radix[i] < rmin ? pl.radix[i] : rmin;
  return pl.L / rmin * rw <= 64 ? 1 : 2;
}
// Dynamic LDS of a generic row-pass block: the twiddle tables and each wave's buffers.
inline size_t row_g_lds_bytes(int M, int rw, int wpb, int nbuf) {
  return (size_t(wpb) * nbuf * M * rw + row_tab_len(2 * M)) * 2 * sizeof(float);
}

// Radices a stage of a mixed-radix transform can have (with_radix).
inline bool radix_ok(int r) {
#define SHS_CASE(RR) if (r == RR) return true;
  SHS_RADICES(SHS_CASE)
#undef SHS_CASE
  return false;
}

// Stage lists worth running for length L, best first: fewest stages (each one costs a trip
// through LDS), then the smallest largest radix (registers, idle lanes); the two best sets
// of radices, each in both orders.  Column transforms may also start with radix 32
// (kFirstRadix).  Empty if L has a prime factor above 23.
inline std::vector<std::vector<int>> stage_lists(int L, bool column) {
  struct Set { std::vector<int> r; bool first; };
  std::vector<Set> sets;
  std::vector<int> cur;
  for (int ns = 2; ns <= 5 && sets.empty(); ++ns) {
    // non-increasing radix lists of ns stages with product L
    auto rec = [&](auto&& self, int rest, int left, int most, bool first) -> void {
      if (left == 0) {
        if (rest == 1) sets.push_back(Set{cur, first});
        return;
      }
      for (int r = most; r >= 2; --r) {
        if (rest % r != 0 || !radix_ok(r)) continue;
        cur.push_back(r);
        self(self, rest / r, left - 1, r, first);
        cur.pop_back();
      }
    };
    rec(rec, L, ns, 24, false);
    if (column && L % kFirstRadix == 0 && sets.empty()) {
      cur.push_back(kFirstRadix);
      rec(rec, L / kFirstRadix, ns - 1, 24, true);
      cur.pop_back();
    }
  }
  std::stable_sort(sets.begin(), sets.end(), [](const Set& a, const Set& b) {
    return *std::max_element(a.r.begin(), a.r.end()) < *std::max_element(b.r.begin(), b.r.end());
  });
  if (sets.size() > 2) sets.resize(2);
  std::vector<std::vector<int>> out;
  for (const Set& t : sets) {
    out.push_back(t.r);
    std::vector<int> rev = t.r;
    std::reverse(rev.begin() + (t.first ? 1 : 0), rev.end());
    if (rev != t.r) out.push_back(rev);
  }
  return out;
}

// Plan of the stages `rs` (in this order; their product is L).
inline bool fft_plan_from(int L, const std::vector<int>& rs, FftPlan& pl, bool column) {
  for (size_t i = 0; i < rs.size(); ++i)
    if (!radix_ok(rs[i]) && !(column && i == 0 && rs[i] == kFirstRadix)) return false;
  pl = FftPlan{};
  pl.L = L;
  long long prod = 1;
  for (int r : rs) prod *= r;
  if (rs.size() < 2 || prod != L || int(rs.size()) > kMaxStages) return false;
  pl.ns = int(rs.size());
  int ns = 1;
  for (int i = 0; i < pl.ns; ++i) {
    pl.radix[i] = rs[i];
    // x / ns = (umulhi(x, mag) + x) >> sh with sh = ceil(log2 ns), mag = floor(2^32 (2^sh - ns) / ns) + 1;
    // exact for every ns <= 2048 and x < 2^21 (x < L * strip width here)
    int sh = 0;
    while ((1 << sh) < ns) ++sh;
    pl.sh[i] = sh;
    pl.mag[i] = ns == 1 ? 0u : unsigned((((unsigned long long)1 << 32) * ((1ull << sh) - ns)) / ns + 1);
    ns *= rs[i];
  }
  return true;
}

// The row transforms of one stage list: the inverse runs it as it is, the forward reversed.
inline bool row_plans_from(int M, const std::vector<int>& rs, FftPlan& inv, FftPlan& fwd) {
  return fft_plan_from(M, rs, inv, false) && fft_plan_from(M, std::vector<int>(rs.rbegin(), rs.rend()), fwd, false);
}

// A plan's schedule: rows per wave and waves per block of the row pass, filters per synthesis work
// item, stage lists of the row and the column transform.
struct TuneCfg {
  int rw = 1, wpb = 4, fc_syn = 1;
  std::vector<int> prow, pcol;
};

// Whether the row pass of side n can run rw rows per wave and wpb waves per block with the stage
// list `rows`: a block's rows divide N and its LDS stays within the limit; one wave per block only
// where four rows per wave would not otherwise fit.
inline bool row_shape_ok(int n, int rw, int wpb, const std::vector<int>& rows) {
  FftPlan pr, pf;
  if (!(rw == 1 || rw == 2 || rw == 4) || !(wpb == 1 || wpb == 2 || wpb == 4)) return false;
  if (n % (rw * wpb) != 0 || (wpb == 1 && rw < 4)) return false;
  return row_plans_from(n / 2, rows, pr, pf) &&
         row_g_lds_bytes(n / 2, rw, wpb, row_g_bufs(pr, rw)) <= kRowGLdsMax;
}
// Whether the tuner could have chosen schedule c for side n (work items of at most max_run filters).
inline bool schedule_ok(int n, const TuneCfg& c, int max_run) {
  const auto among = [](const std::vector<std::vector<int>>& l, const std::vector<int>& v) {
    return std::find(l.begin(), l.end(), v) != l.end();
  };
  return among(stage_lists(n / 2, false), c.prow) && among(stage_lists(n, true), c.pcol) &&
         row_shape_ok(n, c.rw, c.wpb, c.prow) && c.fc_syn >= 1 && c.fc_syn <= max_run;
}

// ---------------------------------------------------------------- cache file
// One line per schedule: "<version>/<key> <rw> <wpb> <fc_syn> <row radices> <column radices>".
// The version changes with the kernels, their LDS or the stage lists, so that schedules that were
// timed on other kernels are not taken over (files without one hold three-stage lists).
constexpr const char* kScheduleVersion = "v2";
inline std::string join_radices(const std::vector<int>& v, char sep) {
  std::string out;
  for (size_t i = 0; i < v.size(); ++i) out += (i ? std::string(1, sep) : std::string()) + std::to_string(v[i]);
  return out;
}
inline std::vector<int> split_radices(const std::string& t) {
  std::vector<int> v;
  size_t i = 0;
  while (i < t.size()) {
    size_t j = t.find(',', i);
    if (j == std::string::npos) j = t.size();
    v.push_back(std::atoi(t.substr(i, j - i).c_str()));
    i = j + 1;
  }
  return v;
}
inline std::string schedule_line(const std::string& key, const TuneCfg& c) {
  return std::string(kScheduleVersion) + "/" + key + " " + std::to_string(c.rw) + " " + std::to_string(c.wpb) + " " +
         std::to_string(c.fc_syn) + " " + join_radices(c.prow, ',') + " " + join_radices(c.pcol, ',');
}
// The key (without version) and schedule of a line; false for a line of another version or form.
inline bool parse_schedule_line(const char* line, std::string& key, TuneCfg& c) {
  char k[128], prow[128], pcol[128], rest[2];
  if (std::sscanf(line, "%127s %d %d %d %127s %127s %1s", k, &c.rw, &c.wpb, &c.fc_syn, prow, pcol, rest) != 6) return false;
  const std::string full = k, version = std::string(kScheduleVersion) + "/";
  if (full.compare(0, version.size(), version) != 0) return false;
  key = full.substr(version.size());
  c.prow = split_radices(prow);
  c.pcol = split_radices(pcol);
  return true;
}

}  // namespace shs
