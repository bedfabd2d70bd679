// Instantiations of the persistent chunk kernel for one vector type ITER_V,
// panel type ITER_M and tile height ITER_R; the build compiles this file once
// per combination.
#include "iter_tab.h"
#include "dev_persist.h"

#ifndef ITER_V
#error "ITER_V, ITER_M and ITER_R must be defined"
#endif

namespace adef2 {

template <typename V, typename M, int R, int FORM>
static PersistFn<V, M> pick(int KP) {
  switch (KP) {
    case 0: return k_persist<V, M, 0, R, PS_STORED>;
    case 8: return k_persist<V, M, 8, R, FORM>;
    case 16: return k_persist<V, M, 16, R, FORM>;
    case 24: return k_persist<V, M, 24, R, FORM>;
    case 32: return k_persist<V, M, 32, R, FORM>;
    case 40: return k_persist<V, M, 40, R, FORM>;
    case 48: return k_persist<V, M, 48, R, FORM>;
    case 56: return k_persist<V, M, 56, R, FORM>;
    default: return k_persist<V, M, 64, R, FORM>;
  }
}

template <typename V, typename M, int R>
PersistFn<V, M> pick_persist(int KP, int form) {
  if constexpr (sizeof(M) == 4)
    return form == PS_SPEC ? pick<V, M, R, PS_SPEC>(KP) : pick<V, M, R, PS_STORED>(KP);
  else
    return form == PS_FREE ? pick<V, M, R, PS_FREE>(KP) : pick<V, M, R, PS_STORED>(KP);
}

template PersistFn<ITER_V, ITER_M> pick_persist<ITER_V, ITER_M, ITER_R>(int, int);

}  // namespace adef2
