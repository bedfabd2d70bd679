// Instantiations of the persistent tile-major chunk kernel for one register
// layout ITER_E (steps per tile); the build compiles this file once per layout.
#include "iter_tab.h"
#include "dev_persist_tm.h"

#ifndef ITER_E
#error "ITER_E must be defined"
#endif

namespace adef2 {

template <int E>
PersistTmFn pick_persist_tm(int KP) {
  switch (KP) {
    case 8: return k_persist_tm<8, E>;
    case 16: return k_persist_tm<16, E>;
    case 24: return k_persist_tm<24, E>;
    case 32: return k_persist_tm<32, E>;
    case 40: return k_persist_tm<40, E>;
    case 48: return k_persist_tm<48, E>;
    case 56: return k_persist_tm<56, E>;
    default: return k_persist_tm<64, E>;
  }
}

template PersistTmFn pick_persist_tm<ITER_E>(int);

}  // namespace adef2
