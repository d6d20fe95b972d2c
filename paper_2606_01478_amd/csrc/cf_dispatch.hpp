// Selection of a kernel variant at run time: calls f(models, ctrl, integ, aero)
// with the selection as integral constants. Variants are compiled in parts, one
// translation unit each (CF_PART), so that they compile in parallel; a part's
// dispatch instantiates and serves only its own.
#pragma once
#include <type_traits>

#include "cf_internal.hpp"
#include "cf_layout.hpp"

#ifndef CF_PART
#define CF_PART 0
#endif

namespace cfk {

template <int V>
using const_int = std::integral_constant<int, V>;

// the part that holds a variant: two parts split by the reduced and the full
// terms; with three or four the mixed-model variants are apart (in one part, or
// reduced and full)
template <int PARTS>
constexpr int part_of(int models, bool aero) {
    if (PARTS == 2 || models != MS_BOTH) return aero ? 1 : 0;
    return PARTS == 3 ? 2 : 2 + (aero ? 1 : 0);
}

template <int PARTS, int MODELS, bool AERO, class F>
hipError_t dispatch_variant(const KernelSel& ks, const F& f) {
    if constexpr (part_of<PARTS>(MODELS, AERO) == CF_PART) {
        using M = const_int<MODELS>;
        using A = const_int<AERO>;
        using E = const_int<EULER>;
        using R = const_int<RK4>;
        const bool rk4 = ks.integ == RK4;
        // identified worlds have no onboard controller
        const int ctrl = MODELS == MS_ID ? CTRL_ROTOR : ks.ctrl;
        switch (ctrl) {
            case CTRL_ROTOR: {
                using C = const_int<CTRL_ROTOR>;
                return rk4 ? f(M{}, C{}, R{}, A{}) : f(M{}, C{}, E{}, A{});
            }
            default: break;
        }
        if constexpr (MODELS != MS_ID) {
            switch (ctrl) {
                case CTRL_PID: {
                    using C = const_int<CTRL_PID>;
                    return rk4 ? f(M{}, C{}, R{}, A{}) : f(M{}, C{}, E{}, A{});
                }
                case CTRL_TORQUE: {
                    using C = const_int<CTRL_TORQUE>;
                    return rk4 ? f(M{}, C{}, R{}, A{}) : f(M{}, C{}, E{}, A{});
                }
                case CTRL_POSITION: {
                    using C = const_int<CTRL_POSITION>;
                    return rk4 ? f(M{}, C{}, R{}, A{}) : f(M{}, C{}, E{}, A{});
                }
                default: break;
            }
        }
    }
    return hipErrorInvalidValue;
}

template <int PARTS, class F>
hipError_t dispatch(const KernelSel& ks, const F& f) {
    if (ks.models == MS_FP)
        return ks.aero ? dispatch_variant<PARTS, MS_FP, true>(ks, f) : dispatch_variant<PARTS, MS_FP, false>(ks, f);
    if (ks.models == MS_ID)
        return ks.aero ? dispatch_variant<PARTS, MS_ID, true>(ks, f) : dispatch_variant<PARTS, MS_ID, false>(ks, f);
    if (ks.models == MS_BOTH)
        return ks.aero ? dispatch_variant<PARTS, MS_BOTH, true>(ks, f) : dispatch_variant<PARTS, MS_BOTH, false>(ks, f);
    return hipErrorInvalidValue;
}

// calls g(part) for the part that holds the selection
template <int PARTS, class G>
auto in_part(const KernelSel& ks, const G& g) {
    switch (part_of<PARTS>(ks.models, ks.aero != 0)) {
        case 0: return g(const_int<0>{});
        case 1: return g(const_int<1>{});
        case 2: return g(const_int<PARTS == 2 ? 1 : 2>{});
        default: return g(const_int<PARTS - 1>{});
    }
}

}  // namespace cfk
