// The recurrence of a stack of LSTM layers as one launch per direction (pf_lstm_persist.hip).
#pragma once

#include "pf_common.h"

namespace pf {

struct LstmGeom {
    int T, B, h, r, G, gr, L;
};
// One layer.  Forward writes h_all, c_all, gates, Th and (above the first layer, whose Tx it reads) Tx; backward reads them and
// writes dz, dTh, (above the first layer) dTx, dh0 and dc0.
struct LstmRunLayer {
    const float *Vx, *Ux, *Vh, *Uh, *bias, *h0, *c0, *dhT, *dcT; // bias, dhT, dcT nullable
    float *h_all, *c_all, *gates, *Tx, *Th;
    float *dh0, *dc0, *dz, *dTh, *dTx;
};
struct LstmRecurrence {
    size_t (*floats)(const LstmGeom &g, bool bwd); // workspace that a call should have for it (0: none)
    bool (*fits)(const LstmGeom &g, bool bwd, size_t room); // this device can hold the launch's workgroups at once, and `room` floats do
    // ws: 256-byte aligned; dh_top: gradient of the top layer's outputs, backward only
    int (*run)(const LstmGeom &g, const LstmRunLayer *l, const float *dh_top, bool bwd, float *ws, hipStream_t s);
};
// Members are null where the kernels are not part of the build (host-only builds of the launch schedule).
extern LstmRecurrence lstm_recurrence;
// floats that the workspace of a call has for it
size_t lstm_stack_room(const pf_lstm_stack_desc *d, bool bwd);

} // namespace pf
