// kt_trace_w3.hip -- the trace kernels of kt_trace.hip again, in namespace
// kt_w3, built for 3 waves per SIMD.
//
// Built as kt_trace.hip is, constants of the polynomial series and of the
// steppers stay in vector registers across the step loop, by hand and by the
// compiler's machine loop-invariant code motion; the kernels then need 201 to
// 256 VGPRs and run 2 waves per SIMD.  This file is compiled with that pass off
// (-mllvm -disable-machine-licm, set by the build) and the staged series'
// constants in scalar registers: the others are set up by the scalar unit where
// they are used, ~65 more scalar instructions per step, and the kernels need 118
// to 168 VGPRs, so 3 waves fit on a SIMD with no spills.  The third wave keeps
// the VALU busy on every issue slot, but each ray then takes longer in wall time,
// and the end of a persistent launch waits for the last rays; in this build each
// wave also cycles its priority (kt_trace.hip) so that the oldest waves do not
// take most of the issue slots.  The host picks this form from 32 rays per lane
// of a one-wave grid on (or when a launch shape asks for 3 or more waves per
// SIMD): 2048x2048 disk 39.0 ms against 39.6, 1024x1024 ring 15.4 against 15.0.
#define KT_TRACE_ONLY 1
#define KT_TRACE_NS kt_w3
#define KT_WAVES_PER_EU 3
#include "kt_trace.hip"
