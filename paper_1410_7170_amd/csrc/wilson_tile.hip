// Launch of the Wilson stencil's tile form (wilson_tile.h).
#include "internal.h"
#include "wilson_tile.h"

namespace ovl {

template <int PREC, int NT>
static void wilson_tile_dispatch_n(int mode, bool g5, dim3 grid, const WArgs &a, const Tile &t, const ProArgs &pro,
                                   hipStream_t st, hipEvent_t e0, hipEvent_t e1)
{
    const dim3 b(NT);
    if (g5) {
        switch (mode) {
        case W_PLAIN: launch_k(k_wilson_tile<PREC, W_PLAIN, true, NT>, grid, b, st, e0, e1, a, t, pro); break;
        case W_NORM: launch_k(k_wilson_tile<PREC, W_NORM, true, NT>, grid, b, st, e0, e1, a, t, pro); break;
        case W_SHIFT: launch_k(k_wilson_tile<PREC, W_SHIFT, true, NT>, grid, b, st, e0, e1, a, t, pro); break;
        case W_RUPDATE: launch_k(k_wilson_tile<PREC, W_RUPDATE, true, NT>, grid, b, st, e0, e1, a, t, pro); break;
        case W_RUPDATE0: launch_k(k_wilson_tile<PREC, W_RUPDATE0, true, NT>, grid, b, st, e0, e1, a, t, pro); break;
        case W_SNORM: launch_k(k_wilson_tile<PREC, W_SNORM, true, NT>, grid, b, st, e0, e1, a, t, pro); break;
        case W_LZ1:
        case W_LZ2:
        case W_LZ3:
            if constexpr (PREC == P_F64) {
                if (mode == W_LZ1) launch_k(k_wilson_tile<PREC, W_LZ1, true, NT>, grid, b, st, e0, e1, a, t, pro);
                else if (mode == W_LZ2) launch_k(k_wilson_tile<PREC, W_LZ2, true, NT>, grid, b, st, e0, e1, a, t, pro);
                else launch_k(k_wilson_tile<PREC, W_LZ3, true, NT>, grid, b, st, e0, e1, a, t, pro);
            }
            break;
        default: launch_k(k_wilson_tile<PREC, W_RESNORM, true, NT>, grid, b, st, e0, e1, a, t, pro); break;
        }
    } else {
        launch_k(k_wilson_tile<PREC, W_PLAIN, false, NT>, grid, b, st, e0, e1, a, t, pro);
    }
}

template <int PREC>
static void wilson_tile_dispatch(int mode, bool g5, dim3 grid, const WArgs &a, const Tile &t, const ProArgs &pro,
                                 hipStream_t st, hipEvent_t e0, hipEvent_t e1)
{
    if (t.nt == 512) wilson_tile_dispatch_n<PREC, 512>(mode, g5, grid, a, t, pro, st, e0, e1);
    else wilson_tile_dispatch_n<PREC, 256>(mode, g5, grid, a, t, pro, st, e0, e1);
}

hipError_t launch_wilson_tile(int prec, int mode, bool g5, dim3 grid, const WArgs &a, const Tile &t,
                              const ProArgs &pro, hipStream_t st, hipEvent_t e0, hipEvent_t e1)
{
    if (prec == P_F64) wilson_tile_dispatch<P_F64>(mode, g5, grid, a, t, pro, st, e0, e1);
    else wilson_tile_dispatch<P_F48>(mode, g5, grid, a, t, pro, st, e0, e1);
    return hipGetLastError();
}

}  // namespace ovl
