// Instantiations of the sweep with the two-plane fp32 networks (TUNER_ALGO_AUTO): factored first
// layer, and fp32 matrix first layers in front of a two-plane second layer.
#include "net_split.h"
#include "sweep_kernel.h"

namespace tuner {

#define TUNER_FACTORED(NT1, NT2, NW) {NET_F32_SPLIT, -1, NT1, NT2, 2, NW, 32, sweep_kernel<FactoredNet<NT1, NT2>, 2, NW>}
#define TUNER_FACTORED_ALL(NT1) TUNER_FACTORED(NT1, 0, 16), TUNER_FACTORED(NT1, 1, 16), TUNER_FACTORED(NT1, 2, 16), TUNER_FACTORED(NT1, 3, 8), TUNER_FACTORED(NT1, 4, 8)
#define TUNER_FACTORED_SHARED(NT1) {NET_F32_SPLIT, -3, NT1, 0, 2, 16, 32, sweep_kernel<FactoredNet<NT1, 0, false, true>, 2, 16>}
#define TUNER_SPLIT(KS, NT, NW) {NET_F32_SPLIT, KS, NT, NT, 2, NW, 32, sweep_kernel<SplitNet<F32Net<KS, NT, NT>, NT, NT>, 2, NW>}
#define TUNER_SPLIT_H(KS, NT, NW) {NET_F32_SPLIT, 100 + KS, NT, NT, 2, NW, 32, sweep_kernel<SplitNet<F32HNet<KS, NT, NT>, NT, NT>, 2, NW>}
static const Variant kSplitVariants[] = {
    TUNER_FACTORED_ALL(1), TUNER_FACTORED_ALL(2), TUNER_FACTORED_ALL(3), TUNER_FACTORED_ALL(4),
    // the first layer's tables in memory: 128 x 128 weights fill the two stage buffers
    {NET_F32_SPLIT, -2, 4, 4, 2, 8, 32, sweep_kernel<FactoredNet<4, 4, true>, 2, 8>},
    // rows shared by the workgroup (one hidden layer)
    TUNER_FACTORED_SHARED(1), TUNER_FACTORED_SHARED(2), TUNER_FACTORED_SHARED(3), TUNER_FACTORED_SHARED(4),
    TUNER_SPLIT(2, 1, 16), TUNER_SPLIT(4, 1, 16), TUNER_SPLIT(6, 1, 16), TUNER_SPLIT(8, 1, 16), TUNER_SPLIT(10, 1, 16), TUNER_SPLIT(12, 1, 16), TUNER_SPLIT(14, 1, 16), TUNER_SPLIT(16, 1, 16),
    TUNER_SPLIT(2, 2, 16), TUNER_SPLIT(4, 2, 16), TUNER_SPLIT(6, 2, 16), TUNER_SPLIT(8, 2, 16), TUNER_SPLIT(10, 2, 16), TUNER_SPLIT(12, 2, 16), TUNER_SPLIT(14, 2, 16), TUNER_SPLIT(16, 2, 16),
    TUNER_SPLIT(2, 4, 8), TUNER_SPLIT(4, 4, 8), TUNER_SPLIT(6, 4, 8), TUNER_SPLIT(8, 4, 8), TUNER_SPLIT(10, 4, 8), TUNER_SPLIT(12, 4, 8), TUNER_SPLIT(14, 4, 8), TUNER_SPLIT(16, 4, 8),
    TUNER_SPLIT_H(1, 1, 16), TUNER_SPLIT_H(2, 1, 16), TUNER_SPLIT_H(3, 1, 16), TUNER_SPLIT_H(4, 1, 16),
    TUNER_SPLIT_H(1, 2, 16), TUNER_SPLIT_H(2, 2, 16), TUNER_SPLIT_H(3, 2, 16), TUNER_SPLIT_H(4, 2, 16),
    TUNER_SPLIT_H(1, 4, 8), TUNER_SPLIT_H(2, 4, 8), TUNER_SPLIT_H(3, 4, 8), TUNER_SPLIT_H(4, 4, 8),
};

const Variant* find_variant_split(const Shape& sh) {
  const int key = sh.span ? (sh.table_words ? -2 : sh.rows_shared ? -3 : -1) : (sh.hoist ? 100 + sh.KS : sh.KS);
  for (const Variant& v : kSplitVariants)
    if (v.KS == key && v.NT1 == sh.NT1 && v.NT2 == sh.NT2) return &v;
  return nullptr;
}

}  // namespace tuner
