// soma_rec.hip -- the instances of the exchange recurrence (k_rec_xchg), in a
// translation unit of their own: they take as long to compile as the rest of
// the library.
#include "soma_rec.hpp"
#include "soma_xchg.hpp"

namespace soma {

namespace {

template <bool kRad, bool kL1>
const void* instance(int nch) {
  switch (nch) {
    case 2: return reinterpret_cast<const void*>(&k_rec_xchg<2, kRad, kL1, false>);
    case 3: return reinterpret_cast<const void*>(&k_rec_xchg<3, kRad, kL1, false>);
    case 4: return reinterpret_cast<const void*>(&k_rec_xchg<4, kRad, kL1, false>);
    case 5: return reinterpret_cast<const void*>(&k_rec_xchg<5, kRad, kL1, false>);
    case 6: return reinterpret_cast<const void*>(&k_rec_xchg<6, kRad, kL1, false>);
    case 7: return reinterpret_cast<const void*>(&k_rec_xchg<7, kRad, kL1, false>);
    case 8: return reinterpret_cast<const void*>(&k_rec_xchg<8, kRad, kL1, false>);
    case 9: return reinterpret_cast<const void*>(&k_rec_xchg<9, kRad, kL1, false>);
    case 10: return reinterpret_cast<const void*>(&k_rec_xchg<10, kRad, kL1, false>);
    case 11: return reinterpret_cast<const void*>(&k_rec_xchg<11, kRad, kL1, false>);
    default: return nullptr;
  }
}

}  // namespace

const void* xchg_kernel_for(int H, bool rademacher, bool layer1) {
  const int nch = H / 64;
  if (layer1) return rademacher ? instance<true, true>(nch) : instance<false, true>(nch);
  return rademacher ? instance<true, false>(nch) : instance<false, false>(nch);
}

const void* xchg_pre_kernel_for(int H) {
  switch (H / 64) {
    case 1: return reinterpret_cast<const void*>(&k_rec_xchg<1, false, false, true>);
    case 2: return reinterpret_cast<const void*>(&k_rec_xchg<2, false, false, true>);
    case 3: return reinterpret_cast<const void*>(&k_rec_xchg<3, false, false, true>);
    case 4: return reinterpret_cast<const void*>(&k_rec_xchg<4, false, false, true>);
    case 5: return reinterpret_cast<const void*>(&k_rec_xchg<5, false, false, true>);
    case 6: return reinterpret_cast<const void*>(&k_rec_xchg<6, false, false, true>);
    case 7: return reinterpret_cast<const void*>(&k_rec_xchg<7, false, false, true>);
    case 8: return reinterpret_cast<const void*>(&k_rec_xchg<8, false, false, true>);
    default: return nullptr;
  }
}

}  // namespace soma
