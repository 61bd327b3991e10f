// Host-side choices and checks around the pair launch, on the CPU: the
// library's host source is included to reach them.
#include "../../paper_1911_08275_amd/csrc/api.hip"

#include <cstdio>
#include <cstdlib>

using namespace cp;

static int g_fail = 0;
#define CHECK(c)                                                      \
  do {                                                                \
    if (!(c)) {                                                       \
      printf("check failed at line %d: %s\n", __LINE__, #c);          \
      g_fail = 1;                                                     \
    }                                                                 \
  } while (0)

// A launch of no more items than waves that left one out must not pass, nor one
// with a short queue.
static void check_drained() {
  static unsigned long long st[kStatWords];
  const int64_t waves = 1000;
  for (int64_t n : {(int64_t)1, (int64_t)7, waves}) {
    memset(st, 0, sizeof(st));
    CHECK(!drained(st, n, waves));
    st[5] = (unsigned long long)n - 1;
    CHECK(!drained(st, n, waves));
    st[5] = (unsigned long long)n;
    CHECK(drained(st, n, waves));
  }
  memset(st, 0, sizeof(st));
  CHECK(drained(st, 0, waves));
  const int64_t n = waves + 3;
  for (int k = 0; k < kQueues; k++)
    st[kStatWords - (kQueues - k) * kQStride] = (unsigned long long)(n * (k + 1) / kQueues - n * k / kQueues);
  CHECK(drained(st, n, waves));
  st[kStatWords - kQStride]--;
  CHECK(!drained(st, n, waves));
}

// Waves are tuned where the launch takes them: not for single w_p calls.
static void check_tuned_waves() {
  Call c{};
  c.mode = WP;
  CHECK(!tunes_waves(c));
  c.per_wave = true;
  CHECK(tunes_waves(c));
  c.mode = XI;
  c.per_wave = false;
  CHECK(tunes_waves(c));
  for (bool waves : {false, true}) {
    int calls = 0, two = 0;
    const TuneTimer t = [&](const int *, int, int wv, double &ms) {
      calls++;
      two += wv == 2;
      ms = wv == 2 ? 1.0 : 2.0;   // two waves look faster
      return CP_OK;
    };
    TuneChoice best;
    CHECK(tune_with(t, waves ? "with" : "without", best, waves) == CP_OK);
    CHECK(two == (waves ? 1 : 0) && best.waves == (waves ? 2 : 4));
    CHECK(calls == 7 + 2 + two);
  }
}

// Every number of copies that the default may choose can be asked for.
static void check_copies() {
  for (bool shared : {false, true})
    for (int c = 1; c <= 64; c++) {
      setenv("CP_WP_COPIES", std::to_string(c).c_str(), 1);
      const int got = wp_copies(WP, F32R, 0, 100, 100, 14, 40, 0, 0, shared);
      unsetenv("CP_WP_COPIES");
      const int own = wp_copies(WP, F32R, 0, 100, 100, 14, 40, 0, 0, shared);
      const bool power = !(c & (c - 1));
      CHECK(got == (power && c <= (shared ? 32 : 8) ? c : own));
    }
  CHECK(wp_copies(WP, F32R, 0, 100, 100, 1, 1, 0, 0, true) == 32);
}

// By position every item goes to one wave, in order and in shares.
static void check_positions() {
  for (int64_t grid : {8, 256, 1280, 1792})
    for (int nw = 1; nw <= 4; nw++)
      for (bool share : {false, true}) {
        const int64_t most = position_items(grid, nw);
        for (int64_t n : {(int64_t)1, (int64_t)2, (int64_t)7, (int64_t)65, most / 3, most - 1, most}) {
          if (n < 1 || n > most) continue;
          std::vector<int> got(n, 0);
          for (int64_t b = 0; b < grid; b++) {
            const ItemRun r = position_run(n, b, nw, share);
            CHECK(r.end <= r.begin + nw && r.end <= n);
            for (int64_t i = r.begin; i < r.end; i++) got[i]++;
          }
          CHECK(std::count(got.begin(), got.end(), 1) == n);
        }
      }
  CHECK(position_items(12, 4) == 0);
}

int main() {
  check_positions();
  check_drained();
  check_copies();
  check_tuned_waves();
  if (!g_fail) printf("launch checks passed\n");
  return g_fail;
}
