// process.hpp -- descriptor of a generated process, shared by the generated kernels and the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace me {

// The colour sum inside the amplitude kernel (processes with fused_colour): the operand tables
// of the separate colour-sum kernel of the same form.  With a FusedColour the kernel writes
// D |M_h|^2 as doubles to ((double*)jamp)[row * n_evt + event] instead of the jamps.
struct FusedColour {
    const void* aop;     // FP64 numerators (FP64 kernels of up to six flows) or FP16 / BF16 hi tiles (FP32 kernel)
    const void* aop_lo;  // BF16 lo tiles (BF16 form)
    uint64_t lo_mask;    // tiles with a non-zero lo part (BF16 form)
    int form;            // ME_FP64, ME_MIXED_FP16 or ME_MIXED_BF16 (me.h)
    // processes with hel_sum_in_kernel or lane_min_f64 / lane_min_mixed: if hsum_out is set, the kernel also
    // sums the good helicities (one workgroup holding all of an event block's, or one lane per
    // event for batches of at least that size, or in FP64 the forms of rec_*.hip), in groups of hel_per_group from the first
    // (the order of the separate helicity-sum kernel), times hsum_scale, into hsum_out[event];
    // nothing goes to the jamp scratch
    double* hsum_out;
    double hsum_scale;
    int hel_per_group;
    // processes with flow_weights_in_kernel: if set, the kernel also writes for every group of
    // HelicityGroups::table sum |J_f|^2 over the good helicities of the group, [group][flow][event]
    double* flow_weights = nullptr;
};

// The good helicities of a process with FP64 recursion, two by two.  Tree amplitudes of QED and QCD with
// real couplings and masses obey J_f(-h) = phase conj(J_f(h)) for the combination -h of opposite
// helicities, the phase common to all flows (reversing a helicity conjugates the polarisation vectors
// and spinors, up to sign; the Feynman rules are real in a Majorana basis).  So |M|^2, the flow weights
// and the channel weights of h and -h are equal, and one of the two is evaluated: a row of the jamps,
// |M_h|^2 or channel sums per pair.  The pair is evaluated at the helicity of particle 0 being -.
// All on the device:
// table: n groups of 5 for the kernels whose workgroup evaluates the four quark spin configurations of
//   one gluon configuration: the gluons' signs (bit i: gluon i has helicity +), then the row of the
//   quark spins (-,-), (-,+), (+,-), (+,+), or -1 where neither helicity of that pair is good
// row: for each helicity combination with particle 0 at - (the lower half) its row, or -1; then for
//   each of them how many good helicities the row stands for (0, 1 or 2)
// members: of each row the two helicities' indices among the good ones, -1 where not good
// hel: of each row the signs of the evaluated combination
struct HelicityGroups {
    const int* table;
    int n;
    const int* row;
    const int2* members;
    const signed char* hel;
    int n_rows;   // 0: no recursion, a row is a good helicity (members is null)
};
// how many good helicities row r stands for; PAIRS: whether the rows are pairs (else members is null)
template <bool PAIRS = true>
__device__ __forceinline__ double members_of(const int2* __restrict__ members, int r)
{
    if constexpr (!PAIRS) return 1.0;
    const int2 m = members[r];
    return (m.x >= 0 ? 1.0 : 0.0) + (m.y >= 0 ? 1.0 : 0.0);
}

// The jamps jamp[row][2 flow + re/im][ld]; a row is a good helicity, or a pair of them (HelicityGroups).
// chan: null, or chan[n_evt] channel ids, for which the per-lane single-diagram sums (channel, all) go to
// sde[row][2][ld].  fc: null, or the fused colour sum (then chan must be null, but for channel_in_kernel)
typedef hipError_t (*amp_launch_f64)(const double* mom, int64_t n_evt, int64_t ld, const signed char* hel,
                                     int n_good, double mt, double g, double* jamp, const int* chan, double* sde,
                                     const FusedColour* fc, const HelicityGroups& hg, hipStream_t st);
typedef hipError_t (*amp_launch_f32)(const double* mom, int64_t n_evt, int64_t ld, const signed char* hel,
                                     int n_good, double mt, double g, float* jamp, const int* chan, double* sde,
                                     const FusedColour* fc, const HelicityGroups& hg, hipStream_t st);

struct ProcessDesc {
    const char* name;
    int npar;          // particles, incoming first
    int nc;            // colour flows (jamps)
    int nhel;          // helicity combinations, 2^npar
    int avg;           // initial-state spin x colour average
    int sym;           // identical final-state particle factor (reported, not applied)
    int coupling;      // 0: alpha_em (QED), 1: alpha_s (QCD)
    const int* colour_num;     // nc x nc integer numerators of the colour matrix
    int colour_den;            // their common denominator
    const int* final_massive;  // npar-2 flags: final-state particle carries the top mass
    const int* orderings;      // nc x n_order: the gluon order of each colour flow
    int n_order;               // entries per flow (gluons of the quark line; for gg->gg the three non-root gluons)
    int n_diagrams;            // Feynman diagrams
    int n_amplitudes;          // vertex contractions (four-gluon vertices count 3)
    double flops_lane;         // algorithmic flops of the amplitude kernel per (event, helicity)
    double flops_exec_lane;    // flops it executes (more when segments recompute currents)
    double flops_recursion;    // FP64 recursion: flops of an event's jamps, and of the colour sum of a row (0: none)
    double flops_colour_row;
    int nslot;                 // partial jamp slots per (event, helicity); 0: jamps written directly
    const int* diagram_lines;  // n_diagrams x lines_per_diagram internal-line masks (0-padded)
    int lines_per_diagram;
    int sde_supported;         // single-diagram channel weights available
    int fused_colour;          // the amplitude kernels can do the colour sum themselves (FusedColour)
    int hel_sum_in_kernel;     // ... and the helicity sum (FusedColour.hsum_out; at most 16 good helicities)
    // batches from this size take the kernel with one lane per event, which also sums the helicities
    // (0: none): FP64, and mixed forms (of one flow)
    int64_t lane_min_f64, lane_min_mixed;
    int64_t (*aux_doubles)(int n_rows);  // doubles per event that the FP64 launch needs after the jamps (null: none)
    int channel_in_kernel;     // the FP64 kernel that sums the helicities also applies the channel weight (chan with fc)
    int rows_in_kernel;        // the FP64 kernel writes D |M_h|^2 of every row (a FusedColour without hsum_out) ...
    int flow_weights_in_kernel;  // ... and the flow weights (FusedColour.flow_weights)
    int recursion;             // the FP64 jamps come from the recursion, without partial slots
    amp_launch_f64 launch_f64;
    amp_launch_f32 launch_f32;
};

// FP64 colour-flow amplitudes by recursion (rec_*.hip); the arguments of launch_f64
namespace rec_ee {
hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const HelicityGroups& hg, double mt, double gs,
                  double* jamp, const int* chan, double* sde, const FusedColour* fc, hipStream_t st);
}
namespace rec2 {
hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const HelicityGroups& hg, double mt, double gs,
                  double* jamp, const int* chan, double* sde, const FusedColour* fc, hipStream_t st);
}
namespace rec3 {
hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const HelicityGroups& hg, double mt, double gs,
                  double* jamp, const int* chan, double* sde, const FusedColour* fc, hipStream_t st);
}
namespace rec4 {
hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const HelicityGroups& hg, double mt, double gs,
                  double* jamp, const FusedColour* fc, hipStream_t st);
}
// gg -> tt~ggg: jamp is followed by aux_doubles(n_rows) doubles per event of the padded batch (ld)
namespace rec5 {
int64_t aux_doubles(int n_rows);
hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const HelicityGroups& hg, double mt, double gs,
                  double* jamp, hipStream_t st);
}

const ProcessDesc* process_ee_mumu();
const ProcessDesc* process_gg_tt();
const ProcessDesc* process_gg_ttg();
const ProcessDesc* process_gg_ttgg();
const ProcessDesc* process_gg_ttggg();
const ProcessDesc* process_gg_gg();
const ProcessDesc* process_ee_mumu_z();

}  // namespace me
