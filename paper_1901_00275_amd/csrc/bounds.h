// Arithmetic that kernels rely on and that is checked on the CPU as well: plain C, no device types.
#pragma once
#include <math.h>
#include <stdint.h>

#ifdef __HIPCC__
#define VLQ_HD __attribute__((host)) __attribute__((device, always_inline)) static inline
#else
#define VLQ_HD static inline
#endif

// ---- places of k_scan_wide (scan_wide.hip) ----
// The points of a workgroup's lists are laid end to end and handed out in turns of SW_TURN places.  A workgroup can
// meet every stored point, up to 2^31 - 1, so the places one past the last turn need the 32nd bit.
#define SW_NT 512              // threads of a workgroup
#define SW_U 4                 // chunks of 64 points per wave and turn
#define SW_TURN (SW_NT * SW_U) // points per workgroup and turn
typedef uint32_t sw_place_t;

VLQ_HD sw_place_t sw_wave_base(sw_place_t turn, int wave) { return turn + (sw_place_t)wave * (64u * SW_U); }
VLQ_HD sw_place_t sw_place(sw_place_t base, int u, int lane) { return base + 64u * (sw_place_t)u + (sw_place_t)lane; }
