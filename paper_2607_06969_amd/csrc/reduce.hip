// reduce.hip -- float64 per-configuration sums of per-atom values.
//
// E_c = sum_i E_i (Eq. 1) and V_c = sum_i W_i (Eq. 4), plus optional
// kinetic energies, are summed in float64 in a fixed order: every
// configuration's caller-order atom range is cut into chunks, one block sums
// a chunk in a fixed shape (wavefront butterflies, then the wavefronts in
// order), and the block that ends a configuration's last chunk sums its chunk
// sums the same way (a second kernel for them costs 4.5 us, what any kernel
// behind another one does).  Results are bitwise reproducible run to run.
#include "reduce.hpp"

namespace nepmi {

// Bound by the two trips through memory (an item's values, then the other
// items' sums).
template <class T>
__global__ __launch_bounds__(kRedThreads) void k_sums(SumArgs<T> a) {
  __shared__ SumShared sh;
  sum_item<kRedThreads>((int)blockIdx.x, a, sh);
}

int Reducer::setup(int n_cfg_, const int64_t* atom_off, Uploader& up) {
  std::vector<RedItem>& items = host_items;
  std::vector<int>& start = host_start;
  items.clear();
  start.assign((size_t)n_cfg_ + 1, 0);
  for (int c = 0; c < n_cfg_; ++c) {
    start[(size_t)c] = (int)items.size();
    int64_t a = atom_off[c];
    const int64_t b = atom_off[c + 1], chunk = red_chunk(b - a);
    do {
      RedItem it;
      it.cfg = c;
      it.a0 = a;
      it.a1 = (b - a > chunk) ? a + chunk : b;
      items.push_back(it);
      a = it.a1;
    } while (a < b);
  }
  start[(size_t)n_cfg_] = (int)items.size();
  host_done.assign((size_t)n_cfg_ + 1, 0);  // the last one counts all items
 
  n_cfg = n_cfg_;
  n_items = (int)items.size();
  int rc;
  if ((rc = up.add(items.data(), sizeof(RedItem) * items.size(), items_dev)) ||
      (rc = up.add(start.data(), 4 * start.size(), start_dev)) ||
      (rc = up.add(host_done.data(), 4 * host_done.size(), done_dev)) ||
      (rc = part.ensure(sizeof(double) * kRedValues * items.size())))
    return rc;
  return NEPMI_OK;
}

template <class T>
int Reducer::run(hipStream_t st, const SumArgs<T>& a) const {
  hipLaunchKernelGGL(k_sums<T>, dim3(a.n_items), dim3(kRedThreads), 0, st, a);
  NEPMI_HIP(hipGetLastError());
  return NEPMI_OK;
}

template int Reducer::run(hipStream_t, const SumArgs<float>&) const;
template int Reducer::run(hipStream_t, const SumArgs<double>&) const;

}  // namespace nepmi
