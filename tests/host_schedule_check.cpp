// Host build of the schedule cache (paper_1112_1805_amd/csrc/schedule.hpp): every schedule the
// tuner can choose survives a trip through a cache line, and every other line or schedule is
// refused.  Prints the failing cases and exits non-zero if there are any.
#include "schedule.hpp"

using namespace shs;

static int bad = 0;
static void expect(bool ok, const std::string& what) {
  if (!ok) { std::printf("FAIL %s\n", what.c_str()); ++bad; }
}

int main() {
  const int kRun = 16;
  long sides = 0, schedules = 0;
  for (int n = 64; n <= kGenericMaxN; n += 8) {
    if ((n & (n - 1)) == 0) continue;
    const auto rows = stage_lists(n / 2, false), cols = stage_lists(n, true);
    if (rows.empty() || cols.empty()) continue;
    ++sides;
    for (const auto& r : rows)
      for (const auto& c : cols)
        for (int rw : {1, 2, 4})
          for (int wpb : {1, 2, 4})
            for (int fc : {1, 16}) {
              if (!row_shape_ok(n, rw, wpb, r)) continue;
              TuneCfg a;
              a.rw = rw; a.wpb = wpb; a.fc_syn = fc; a.prow = r; a.pcol = c;
              const std::string key = "gfx950/n" + std::to_string(n) + "/J3/q2/s0";
              TuneCfg b;
              std::string k;
              const bool ok = parse_schedule_line((schedule_line(key, a) + "\n").c_str(), k, b);
              expect(ok && k == key && b.rw == rw && b.wpb == wpb && b.fc_syn == fc && b.prow == r && b.pcol == c &&
                         schedule_ok(n, b, kRun), schedule_line(key, a));
              ++schedules;
            }
  }
  expect(sides > 60, "sides");
  // lines of another version or form
  TuneCfg c;
  std::string k;
  for (const char* line : {"gfx950/n360/J3/q2/s0 2 4 4 4,5,9 8,5,9\n", "v1/gfx950/n360/J3/q2/s0 2 4 4 12,15 24,15\n",
                           "v2/gfx950/n360/J3/q2/s0 2 4 4 12,15\n", "v2/gfx950/n360/J3/q2/s0 2 4\n",
                           "v2/gfx950/n360/J3/q2/s0 a 4 4 12,15 24,15\n", "v2/gfx950/n360/J3/q2/s0 2 4 4 12,15 24,15 9\n",
                           "", "\n", "v2/"})
    expect(!parse_schedule_line(line, k, c), std::string("line accepted: ") + line);
  // schedules the tuner could not have chosen
  const auto sched = [](int rw, int wpb, int fc, std::vector<int> r, std::vector<int> col) {
    TuneCfg t;
    t.rw = rw; t.wpb = wpb; t.fc_syn = fc; t.prow = std::move(r); t.pcol = std::move(col);
    return t;
  };
  const auto r360 = stage_lists(180, false)[0], c360 = stage_lists(360, true)[0];
  expect(schedule_ok(360, sched(2, 4, 4, r360, c360), kRun), "a valid schedule of 360");
  for (int rw : {-1, 0, 3, 8}) expect(!schedule_ok(360, sched(rw, 4, 4, r360, c360), kRun), "rows per wave");
  for (int wpb : {-4, 0, 3, 8}) expect(!schedule_ok(360, sched(2, wpb, 4, r360, c360), kRun), "waves per block");
  for (int fc : {-1, 0, kRun + 1, 1000}) expect(!schedule_ok(360, sched(2, 4, fc, r360, c360), kRun), "filters per item");
  expect(!schedule_ok(72, sched(4, 4, 1, stage_lists(36, false)[0], stage_lists(72, true)[0]), kRun), "rows of a block");
  for (const auto& r : std::vector<std::vector<int>>{{}, {180}, {4, 5, 9}, {12, 14}, {1, 12, 15}, {36, 5}, {0, 0}, {-12, -15}})
    expect(!schedule_ok(360, sched(2, 4, 4, r, c360), kRun), "row list " + join_radices(r, ','));
  for (const auto& r : std::vector<std::vector<int>>{{}, {8, 5, 9}, {24, 14}, {12, 15}})
    expect(!schedule_ok(360, sched(2, 4, 4, r360, r), kRun), "column list " + join_radices(r, ','));
  // a three-stage list whose two LDS buffers pass the row pass's limit: 67,200 bytes
  expect(!row_shape_ok(480, 4, 4, {16, 3, 5}), "LDS of a row block");
  std::printf("%ld sides, %ld schedules\n%s\n", sides, schedules, bad ? "FAIL" : "OK");
  return bad ? 1 : 0;
}
