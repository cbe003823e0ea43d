"""How matching calls are cut up: no work-group walks far more tiles than the chip's
share of the call, be one set much longer than the other; sets are copied to fp16 only
where their tiles are staged several times (launches recorded on the host)."""
from launch_record import run

DRIVER = r"""
namespace sift {
void set_last_error(const std::string&) {}
static MatchHdr hdr;
static int grid;
hipError_t launch_match_setup(const MatchHdr&, const MatchSetupChunk&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_match_rows(const MatchHdr& h, int, int g, hipStream_t) { hdr = h; grid = g; return hipSuccess; }
hipError_t launch_match_cols(const MatchHdr&, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_match_emit(const MatchHdr&, int, float, hipStream_t) { return hipSuccess; }
}
using sift::hdr;
using sift::grid;
// the plan of n pairs of a x b rows
static void plan(int n, int a, int b) {
  sift_match_pair q;
  std::memset(&q, 0, sizeof q);
  q.desc_a = fake<const float>(1);
  q.desc_b = fake<const float>(2);
  q.cap_a = a;
  q.cap_b = b;
  q.matches = fake<sift_match>(3);
  q.n_matches = fake<int32_t>(4);
  q.capacity = 1;
  std::vector<sift_match_pair> pairs(n, q);
  size_t bytes = 0;
  CHECK(sift_match_workspace_size(n, pairs.data(), &bytes) == SIFT_OK);
  CHECK(sift_match_batch(n, pairs.data(), 0.8f, fake<char>(5), bytes, nullptr) == SIFT_OK);
  const long own = hdr.own_rows, ta = (a + 127) / 128, tb = (b + 127) / 128;
  const long at = (a + own - 1) / own, bt = (b + own - 1) / own;
  const long steps = n * (at * tb + bt * ta), share = steps / 512 > 0 ? steps / 512 : 1;
  // work-groups per pair
  const long groups = grid / n;
  CHECK(grid % n == 0);
  auto parts = [&](long tiles) { return std::min<long>(8, (tiles + share - 1) / share); };
  std::printf("%d x (%d, %d): half %d own %ld: %ld groups a pair, %ld x %ld and %ld x %ld parts wanted\n", n, a, b,
              !!hdr.half, own, groups, at, parts(tb), bt, parts(ta));
  CHECK(groups == at * parts(tb) + bt * parts(ta));
}
#define PLAN(n, a, b, h) do { plan(n, a, b); CHECK(!!hdr.half == h); } while (0)
int main() {
  // one set much longer than the other: walks of one tile, and a few of hundreds
  PLAN(1, 65536, 100, 0);
  PLAN(1, 100, 65536, 0);
  PLAN(2, 60000, 60, 0);
  PLAN(8, 16384, 128, 0);
  PLAN(32, 4096, 128, 0);
  PLAN(1, 65536, 4000, 1);
  // a set whose tiles are each staged once or twice: no copies
  PLAN(200, 1, 5000, 0);
  PLAN(1024, 100, 100, 0);
  PLAN(64, 64, 4000, 0);
  // sets of about equal size
  PLAN(32, 2000, 2000, 1);
  PLAN(8, 2000, 2000, 1);
  PLAN(1, 2000, 2000, 0);
  PLAN(1, 8192, 7900, 1);
  PLAN(1, 300, 263, 0);
  PLAN(1, 1, 1, 0);
  PLAN(1, 65536, 65536, 1);
  return fails;
}
"""


def test_plans(tmp_path):
    run(tmp_path, ["sift_match.cpp"], DRIVER)
