// lbm_plane.hip -- launches of the one-launch D2Q9 step, in a translation unit of their own
// (compiled in parallel with the other passes).
#include "lbm_plane.hpp"

#include "lbm_host.hpp"

namespace lbmh {
namespace {

template <typename T, typename P, bool S, int PH, int TX, int TY, int NT>
void launch(const lbm_solver *h) {
    const uint32_t ntx = (uint32_t)((h->nx + TX - 1) / TX);
    const uint32_t nt = ntx * (uint32_t)((h->ny + TY - 1) / TY);
    const uint32_t per = (nt + 7) / 8;
    hipLaunchKernelGGL((lbm::k_plane_step<T, P, S, PH, TX, TY, NT>), dim3(8 * per), dim3(NT), 0,
                       h->stream, ws_ptr<const P>(h, PH ? h->L.f2 : h->L.f),
                       ws_ptr<P>(h, PH ? h->L.f : h->L.f2), ws_ptr<const T>(h, h->L.eps),
                       ws_ptr<const T>(h, h->L.muD), ws_ptr<const T>(h, h->L.muF), mask_ptr(h),
                       grid_of(h), ntx, nt, per, phys_of<T>(h));
}

// Small tiles have the shortest chain of loads and barriers (with solids every thread forms one
// record, without 144 of the 256 do), and the ring cells computed again cost nothing on an idle
// chip.  On larger planes the ring cells' arithmetic counts and the tile is 32 x 8 (whole 128-byte
// lines in FP32, 1.7 records per cell against 2.25); plane_shape chooses.  us per step, 8 x 8
// against 32 x 8: FP64 channel with walls 128 x 64 7.3 / 11.3, 320 x 160 11.0 / 11.3; FP32 box 200
// x 200 4.9 / 5.8, 256 x 256 6.0 / 5.9, 512 x 512 13.2 / 10.0, 1024 x 1024 39.5 / 27.9; FP64 200 x
// 200 7.6 / 8.0, 256 x 256 9.0 / 8.4 (16 x 16, 64 x 8 and 64 x 16 tiles within 4 % of 32 x 8 on
// large planes, slower on small ones).
template <typename T, typename P, bool S, int PH>
void launch_shape(const lbm_solver *h) {
    if (h->plane == kPlaneSmall) launch<T, P, S, PH, 8, 8, 256>(h);
    else launch<T, P, S, PH, 32, 8, 256>(h);
}

template <typename T, typename P>
void launch_cfg(const lbm_solver *h) {
    if (h->solids) {
        if (h->phase) launch_shape<T, P, true, 1>(h);
        else launch_shape<T, P, true, 0>(h);
    } else {
        if (h->phase) launch_shape<T, P, false, 1>(h);
        else launch_shape<T, P, false, 0>(h);
    }
}

}  // namespace

void launch_plane_step(const lbm_solver *h) {
    switch (h->storage) {
    case LBM_F64: launch_cfg<double, double>(h); break;
    case LBM_F32: launch_cfg<float, float>(h); break;
    case LBM_F16_SHIFTED: launch_cfg<float, _Float16>(h); break;
    default: launch_cfg<float, __bf16>(h); break;
    }
}

}  // namespace lbmh
