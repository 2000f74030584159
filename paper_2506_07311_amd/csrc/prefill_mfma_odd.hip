// Paged prefill on the matrix cores: the kernels of head_dims 80, 96 and 112.
#include "prefill_mfma_impl.h"

namespace pa {

template pa_status launch_prefill_mfma_dim<80>(const AttnArgs&, const prefill::PrefillPlan&, int64_t, int64_t,
                                               hipStream_t);
template pa_status launch_prefill_mfma_dim<96>(const AttnArgs&, const prefill::PrefillPlan&, int64_t, int64_t,
                                               hipStream_t);
template pa_status launch_prefill_mfma_dim<112>(const AttnArgs&, const prefill::PrefillPlan&, int64_t, int64_t,
                                                hipStream_t);

}  // namespace pa
