"""Export of a forest's node arrays when the device has no memory left for the
unpacked slices, on the CPU: the program's own HIP functions copy host memory and
refuse every allocation."""
from tests._native import run_host

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include "internal.h"

extern "C" {
hipError_t hipMalloc(void**, size_t) { return hipErrorOutOfMemory; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
}

int main() {
  // 40 trees: tree t a chain of t splits, its slot 100 nodes long; node words are
  // left child | bin | column, a leaf's column 255 (its value in the other bits)
  constexpr int kTrees = 40, kSlot = 100;
  std::vector<uint64_t> words(kTrees * kSlot);
  std::vector<uint32_t> weight(kTrees * kSlot);
  std::vector<int32_t> n_nodes(kTrees);
  std::vector<int64_t> base(kTrees);
  for (int i = 0; i < kTrees * kSlot; ++i) {
    words[i] = 0x0123456789ull * (uint64_t)(i + 1) & ~0xFFull;
    words[i] |= i % 3 ? 255 : 7;
    weight[i] = i * 7 + 1;
  }
  int total = 0;
  aiwc_rf_forest f;
  f.params.push_back({kTrees, 1, 1, 1, 1});
  f.first_task.push_back(0);
  f.tasks.resize(kTrees);
  for (int t = 0; t < kTrees; ++t) {
    n_nodes[t] = 2 * t + 1;
    base[t] = f.tasks[t].node_base = t * kSlot;
    total += n_nodes[t];
  }
  uint32_t ok = 0;
  f.status_host = &ok;
  f.waited = true;
  f.nodes.p = words.data();
  f.node_N.p = weight.data();
  f.n_nodes.p = n_nodes.data();
  f.node_base.p = base.data();
  auto all = [&](int a, int e, std::vector<uint8_t>& col, std::vector<uint8_t>& bin, std::vector<int32_t>& left,
                 std::vector<int64_t>& q, std::vector<int32_t>& N) {
    col.assign(total, 0); bin.assign(total, 0); left.assign(total, 0); q.assign(total, 0); N.assign(total, 0);
    return aiwc_rf_forest_export_host(&f, 0, a, e, col.data(), bin.data(), left.data(), q.data(), N.data());
  };
  std::vector<uint8_t> col, bin, col1, bin1;
  std::vector<int32_t> left, N, left1, N1;
  std::vector<int64_t> q, q1;
  int rc = all(0, kTrees, col, bin, left, q, N), same = 1, at = 0;
  // against the trees one by one, which are copied without device memory
  for (int t = 0; t < kTrees && rc == 0; ++t) {
    if (all(t, t + 1, col1, bin1, left1, q1, N1) != 0) same = 0;
    for (int i = 0; i < n_nodes[t]; ++i, ++at)
      same &= col[at] == col1[i] && bin[at] == bin1[i] && left[at] == left1[i] && q[at] == q1[i] && N[at] == N1[i];
  }
  // some arrays only
  std::vector<int32_t> only(total, 0);
  const int rc2 = aiwc_rf_forest_export_host(&f, 0, 0, kTrees, nullptr, nullptr, only.data(), nullptr, nullptr);
  std::printf("%d %d %d %d\n", rc, same && at == total, rc2, only == left);
}
"""


def test_export_without_device_memory(tmp_path):
    assert run_host(tmp_path, PROGRAM).split() == ["0", "1", "0", "1"]
