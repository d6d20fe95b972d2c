// Adjoint rollout kernels: their launcher (the kernels and device code are in
// cf_rollout_impl.hpp, shared with the forward's translation units).
#include "cf_rollout_impl.hpp"

namespace cfk {

constexpr int ROLL_PARTS = 4;

// the variants compiled in part P (cf_dispatch.hpp)
template <int P>
hipError_t launch_bwd_part(const KernelSel& ks, const RollArgs& a, const int4* tiles, int n_tiles, hipStream_t s);

template <>
hipError_t launch_bwd_part<CF_PART>(const KernelSel& ks, const RollArgs& a, const int4* tiles, int n_tiles, hipStream_t s) {
    return dispatch<ROLL_PARTS>(ks, [&](auto m, auto c, auto i, auto e) {
        return launch_bwd_t<m(), c(), i(), e() != 0>(ks, a, tiles, n_tiles, s);
    });
}

#if CF_PART == 0
template <> hipError_t launch_bwd_part<1>(const KernelSel&, const RollArgs&, const int4*, int, hipStream_t);
template <> hipError_t launch_bwd_part<2>(const KernelSel&, const RollArgs&, const int4*, int, hipStream_t);
template <> hipError_t launch_bwd_part<3>(const KernelSel&, const RollArgs&, const int4*, int, hipStream_t);

hipError_t launch_rollout_bwd(const KernelSel& ks, const RollArgs& a, const int4* tiles, int n_tiles, hipStream_t s) {
    return in_part<ROLL_PARTS>(ks, [&](auto p) { return launch_bwd_part<p()>(ks, a, tiles, n_tiles, s); });
}
#endif

}  // namespace cfk
