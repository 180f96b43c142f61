// mlp_host.cpp -- workspace layout of the learned initialiser's network.
#include "mlp.hpp"

namespace hf {

constexpr int64_t MlpLayout::kW[4];
constexpr int64_t MlpLayout::kB[4];
constexpr int MlpLayout::kIn[4];
constexpr int MlpLayout::kOutDim[4];

namespace {

struct Carver {
  char* p;
  int64_t used = 0;
  template <class T>
  T* take(int64_t n) {
    const int64_t bytes = (static_cast<int64_t>(sizeof(T)) * n + 255) & ~int64_t(255);
    T* r = p ? reinterpret_cast<T*>(p + used) : nullptr;
    used += bytes;
    return r;
  }
};

MlpWorkspace carve(Carver& c, int B) {
  MlpWorkspace w{};
  for (int l = 0; l < 4; ++l) {
    const int in = MlpLayout::kIn[l], out = MlpLayout::kOutDim[l];
    w.a[l] = c.take<uint16_t>(static_cast<int64_t>(B) * in);
    w.at[l] = c.take<uint16_t>(static_cast<int64_t>(B) * in);
    w.wb[l] = c.take<uint16_t>(static_cast<int64_t>(in) * out);
    w.wt[l] = c.take<uint16_t>(static_cast<int64_t>(in) * out);
    w.dz[l + 1] = c.take<uint16_t>(static_cast<int64_t>(B) * out);
    w.dzt[l + 1] = c.take<uint16_t>(static_cast<int64_t>(B) * out);
    if (l >= 1) w.z[l] = c.take<float>(static_cast<int64_t>(B) * in);
  }
  w.y = c.take<float>(static_cast<int64_t>(B) * kMlpOutPad);
  w.loss_part = c.take<double>(static_cast<int64_t>(B) * kMlpOutPad / 256);
  return w;
}

}  // namespace

int64_t mlp_workspace_bytes(int B) {
  Carver c{nullptr};
  carve(c, B);
  return c.used;
}

MlpWorkspace mlp_carve(void* base, int B) {
  Carver c{static_cast<char*>(base)};
  return carve(c, B);
}

}  // namespace hf
