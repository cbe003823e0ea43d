"""Where the band scan runs: a launch of its own, one work-group per image, unless
bands and images are few.  Images of a few bands each stay far below the bands
that a scan pays for, and one work-group would go through them in turn."""
from launch_record import run

DRIVER = r"""
namespace sift {
static int scans, emits;
hipError_t launch_setup(const HdrPtrs&, const SetupChunk&, hipStream_t) { return hipSuccess; }
hipError_t launch_finalize(const HdrPtrs&, int, const DevParams&, hipStream_t) { return hipSuccess; }
hipError_t launch_blur(const BlurArgs&, int, int, hipStream_t) { return hipSuccess; }
bool chain_supported(int, int, int, const int*) { return false; }
hipError_t launch_chain(const ChainArgs&, int, int, int, const int*, int, hipStream_t) { return hipSuccess; }
hipError_t launch_detect(char*, const HdrPtrs&, int, const DevParams&, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_band_scan(char*, const HdrPtrs&, int, const DevParams&, hipStream_t) { ++scans; return hipSuccess; }
hipError_t launch_emit(char*, const HdrPtrs&, int, const DevParams&, int, hipStream_t) { ++emits; return hipSuccess; }
hipError_t launch_refine(char*, const HdrPtrs&, int, const DevParams&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_orient(char*, const HdrPtrs&, int, const DevParams&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_ori_scan(char*, const HdrPtrs&, int, const DevParams&, hipStream_t) { return hipSuccess; }
hipError_t launch_describe(char*, const HdrPtrs&, int, const DevParams&, int, hipStream_t) { return hipSuccess; }
hipError_t bounds_count_blur(unsigned long long*, bool) { return hipErrorNotSupported; }
hipError_t bounds_count_kernels(unsigned long long*, bool) { return hipErrorNotSupported; }
hipError_t bounds_count_match(unsigned long long*, bool) { return hipErrorNotSupported; }
hipError_t bounds_count_verify(unsigned long long*, bool) { return hipErrorNotSupported; }
}
// scans of one launch sequence of n images of h x w
static int scans(int n, int h, int w, int octaves) {
  sift_params p;
  CHECK(sift_params_default(&p) == SIFT_OK);
  p.n_octaves = octaves;
  p.n_streams = 1;
  p.max_candidates = p.max_keypoints = 64;
  sift_handle* hd = nullptr;
  CHECK(sift_create(&p, &hd) == SIFT_OK);
  std::vector<const float*> im(n, fake<const float>(1));
  std::vector<int32_t> hs(n, h), wd(n, w);
  std::vector<int64_t> pitch(n, w);
  sift_output o;
  std::memset(&o, 0, sizeof o);
  o.keypoints = fake<sift_keypoint>(2);
  o.descriptors = fake<float>(3);
  o.count = fake<int32_t>(4);
  o.capacity = 64;
  std::vector<sift_output> outs(n, o);
  size_t bytes = 0;
  CHECK(sift_batch_workspace_size(hd, n, hs.data(), wd.data(), &bytes) == SIFT_OK);
  sift::scans = sift::emits = 0;
  CHECK(sift_extract_batch(hd, n, im.data(), hs.data(), wd.data(), pitch.data(), fake<char>(5), bytes,
                           outs.data(), nullptr) == SIFT_OK);
  CHECK(sift::emits == 1);
  sift_destroy(hd);
  return sift::scans;
}
int main() {
  CHECK(scans(1, 97, 97, 4) == 0);      // 19 bands
  CHECK(scans(4, 97, 97, 4) == 0);
  CHECK(scans(24, 97, 97, 4) == 1);     // 456 bands
  CHECK(scans(512, 18, 18, 1) == 1);    // a band each
  CHECK(scans(1, 480, 640, 4) == 0);    // 110
  CHECK(scans(1, 2048, 2048, 4) == 0);
  CHECK(scans(1, 4400, 100, 3) == 1);   // beyond 512 bands
  return fails;
}
"""


def test_scan_has_its_own_launch_where_images_are_many(tmp_path):
    run(tmp_path, ["sift_api.cpp"], DRIVER)
