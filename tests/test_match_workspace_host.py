"""Which workspaces a matching call takes: what sift_match_workspace_size asks for and
anything down to the documented least, nothing below (no launch then)."""
from launch_record import run

DRIVER = r"""
namespace sift {
void set_last_error(const std::string&) {}
static int launches;
hipError_t launch_match_setup(const MatchHdr&, const MatchSetupChunk&, int, hipStream_t) { ++launches; return hipSuccess; }
hipError_t launch_match_rows(const MatchHdr&, int, int, hipStream_t) { ++launches; return hipSuccess; }
hipError_t launch_match_cols(const MatchHdr&, int, int, hipStream_t) { ++launches; return hipSuccess; }
hipError_t launch_match_emit(const MatchHdr&, int, float, hipStream_t) { ++launches; return hipSuccess; }
}
static size_t up(size_t v) { return (v + 255) / 256 * 256; }
static void sizes(const std::vector<std::pair<int, int>>& sets) {
  const int n = (int)sets.size();
  std::vector<sift_match_pair> q(n);
  std::memset(q.data(), 0, n * sizeof q[0]);
  size_t least = up(96 * n) + 2 * up(4 * n + 4);
  for (int i = 0; i < n; ++i) {
    const size_t a = sets[i].first, b = sets[i].second;
    q[i].desc_a = fake<const float>(1);
    q[i].desc_b = fake<const float>(2);
    q[i].cap_a = (int)a;
    q[i].cap_b = (int)b;
    q[i].matches = fake<sift_match>(3);
    q[i].n_matches = fake<int32_t>(4);
    q[i].capacity = 1;
    least += up(16 * (a + b));
  }
  size_t asked = 0;
  CHECK(sift_match_workspace_size(n, q.data(), &asked) == SIFT_OK);
  CHECK(least <= asked);
  auto call = [&](size_t bytes) {
    sift::launches = 0;
    const sift_status st = sift_match_batch(n, q.data(), 0.8f, fake<char>(5), bytes, nullptr);
    CHECK((st == SIFT_OK) == (sift::launches > 0));
    return st;
  };
  std::printf("%d pairs, first %d x %d: asked for %zu, least %zu\n", n, sets[0].first, sets[0].second, asked, least);
  CHECK(call(asked) == SIFT_OK && call(least) == SIFT_OK && call((asked + least) / 2) == SIFT_OK);
  CHECK(call(least - 1) == SIFT_ERR_WORKSPACE_TOO_SMALL);
  CHECK(call(least - 256) == SIFT_ERR_WORKSPACE_TOO_SMALL);
}
int main() {
  sizes({{300, 263}});
  sizes({{8192, 7900}});
  sizes({{1, 1}});
  sizes({{0, 50}, {1500, 1700}});
  sizes({{65536, 100}});
  sizes({{100, 65536}});
  sizes(std::vector<std::pair<int, int>>(32, {2000, 2000}));
  sizes(std::vector<std::pair<int, int>>(70, {129, 1025}));
  return fails;
}
"""


def test_sizes_taken_and_refused(tmp_path):
    run(tmp_path, ["sift_match.cpp"], DRIVER)
