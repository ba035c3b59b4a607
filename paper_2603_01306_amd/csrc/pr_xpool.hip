// Exchange areas (pr_xwg.h) for the entry points that have no context: a
// fixed set of slots in device memory per GPU, leased for the length of one
// call, so that calls on several threads and streams never share one and
// nothing is allocated per call.  A call that finds every slot leased brings an
// area of its own and frees it when it ends.
#include <mutex>

#include "pr_internal.h"

namespace pr {
namespace {

constexpr int kSlots = 8;  // slot 0 belongs to pr_prox_noalloc
constexpr int kDevices = 64;

static __device__ uint64_t g_slots[kSlots][kXwgWords];
static __device__ uint32_t g_head[kSlots][2];
static __device__ XResult g_result;  // pr_prox_noalloc's

struct DeviceSlots {
  uint64_t *slots = nullptr;
  uint32_t *head = nullptr;
  XResult *result = nullptr;
  unsigned busy = 0u;  // bit per leased slot
};
std::mutex g_mu;
DeviceSlots g_dev[kDevices];
XResult *g_res = nullptr;  // pinned, kDevices * kSlots entries (written by the kernels)

// Device addresses of this device's slots (looked up once; g_mu held).
bool find_slots(int dev) {
  DeviceSlots &d = g_dev[dev];
  if (d.result) return true;
  void *a = nullptr, *b = nullptr, *c = nullptr;
  if (hipGetSymbolAddress(&a, HIP_SYMBOL(g_slots)) != hipSuccess ||
      hipGetSymbolAddress(&b, HIP_SYMBOL(g_head)) != hipSuccess ||
      hipGetSymbolAddress(&c, HIP_SYMBOL(g_result)) != hipSuccess || !a || !b || !c)
    return false;
  d.slots = static_cast<uint64_t *>(a);
  d.head = static_cast<uint32_t *>(b);
  d.result = static_cast<XResult *>(c);
  return true;
}

}  // namespace

int xwg_cap(hipStream_t s) {
  int cus = 0;
  uint32_t mask[32] = {};
  if (s == hipStreamLegacy) s = nullptr;  // the same stream; the query reads through that handle
  if (hipExtStreamGetCUMask(s, 32, mask) == hipSuccess) {
    for (uint32_t w : mask) cus += __builtin_popcount(w);
  } else {
    (void)hipGetLastError();
  }
  const int cap = cus / 4;
  return cap < 1 ? 1 : (cap < kXwgMax ? cap : kXwgMax);
}

int XLease::take(hipStream_t s, int cap) {
  if (hipGetDevice(&dev_) != hipSuccess || dev_ < 0 || dev_ >= kDevices) return PR_EDEVICE;
  {
    std::lock_guard<std::mutex> lock(g_mu);
    if (!find_slots(dev_)) return PR_EDEVICE;
    if (!g_res &&
        hipHostMalloc((void **)&g_res, sizeof(XResult) * kDevices * kSlots, hipHostMallocPortable) != hipSuccess) {
      g_res = nullptr;
      (void)hipGetLastError();
      return PR_ENOMEM;
    }
    DeviceSlots &d = g_dev[dev_];
    for (int i = 1; i < kSlots; i++) {
      if (d.busy & (1u << i)) continue;
      d.busy |= 1u << i;
      slot_ = i;
      xb = XBuf{d.slots + (size_t)i * kXwgWords, d.head + 2 * i, nullptr, cap};
      res = g_res + dev_ * kSlots + i;
      break;
    }
  }
  if (slot_ == 0) {
    if (hipMalloc((void **)&own_, sizeof(uint64_t) * (kXwgWords + 1)) != hipSuccess) {
      own_ = nullptr;
      (void)hipGetLastError();
      return PR_ENOMEM;
    }
    if (hipHostMalloc((void **)&res, sizeof(XResult), hipHostMallocPortable) != hipSuccess) {
      res = nullptr;
      (void)hipGetLastError();
      return PR_ENOMEM;
    }
    if (hipMemsetAsync(own_, 0, sizeof(uint64_t) * (kXwgWords + 1), s) != hipSuccess) return PR_EDEVICE;
    xb = XBuf{own_, reinterpret_cast<uint32_t *>(own_ + kXwgWords), nullptr, cap};
  }
  *res = XResult{{0.0, 0.0}, 1, 0, -1};
  xb.lost = &res->lost;
  return PR_OK;
}

XLease::~XLease() {
  if (slot_) {
    std::lock_guard<std::mutex> lock(g_mu);
    g_dev[dev_].busy &= ~(1u << slot_);
    return;
  }
  if (own_) {
    (void)hipFree(own_);
    if (res) (void)hipHostFree(res);
  }
}

int xpool_noalloc(XBuf *xb, XResult **res, int cap) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return PR_EDEVICE;
  std::lock_guard<std::mutex> lock(g_mu);
  if (!find_slots(dev)) return PR_EDEVICE;
  *xb = XBuf{g_dev[dev].slots, g_dev[dev].head, &g_dev[dev].result->lost, cap};
  *res = g_dev[dev].result;
  return PR_OK;
}

}  // namespace pr
