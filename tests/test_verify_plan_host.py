"""Verification prepares all pairs of a call in one launch, be they more than a launch's
arguments hold (launches recorded on the host)."""
from launch_record import run

DRIVER = r"""
namespace sift {
void set_last_error(const std::string&) {}
static int setups, entries, preps, prepared;
hipError_t launch_verify_setup(const VerifyHdr&, const VerifySetupChunk& c, hipStream_t) { ++setups; entries += c.count; return hipSuccess; }
hipError_t launch_verify_prep(const VerifyHdr&, int n, hipStream_t) { CHECK(entries == n); ++preps; prepared = n; return hipSuccess; }
hipError_t launch_verify_models(const VerifyHdr&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_verify_hyp(const VerifyHdr&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_verify_refine(const VerifyHdr&, int, hipStream_t) { return hipSuccess; }
}
static void call(int n) {
  sift_verify_pair q;
  std::memset(&q, 0, sizeof q);
  q.kp_a = fake<const sift_keypoint>(1);
  q.kp_b = fake<const sift_keypoint>(2);
  q.matches = fake<const sift_match>(3);
  q.cap = 50;
  q.H = fake<double>(4);
  q.score = fake<double>(5);
  q.n_inliers = fake<int32_t>(6);
  std::vector<sift_verify_pair> pairs(n, q);
  size_t bytes = 0;
  CHECK(sift_verify_workspace_size(n, pairs.data(), 100, &bytes) == SIFT_OK);
  sift::setups = sift::entries = sift::preps = sift::prepared = 0;
  CHECK(sift_verify_batch(n, pairs.data(), fake<const float>(7), 100, 2.0f, 5, fake<char>(8), bytes, nullptr) == SIFT_OK);
  std::printf("%d pairs: %d table launches, %d preparations\n", n, sift::setups, sift::preps);
  CHECK(sift::entries == n);
}
int main() {
  for (int n : {1, 24}) {   // one launch for table and preparation
    call(n);
    CHECK(sift::setups == 1 && sift::preps == 0);
  }
  for (int n : {25, 48, 49, 1024, 4096}) {
    call(n);
    CHECK(sift::preps == 1 && sift::prepared == n);
  }
  return fails;
}
"""


def test_one_preparation(tmp_path):
    run(tmp_path, ["sift_verify.cpp"], DRIVER)
