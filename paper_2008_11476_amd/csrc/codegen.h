// Kernels generated for one fused group and compiled at run time.
//
// The tile interpreter (k_generic) runs any verified group but decides every
// operator, format, border and window offset per pixel.  The source-to-source
// step of Section 6 instead emits a kernel per fused group in which all of
// these are constants: here the group's program is written out as HIP
// source, compiled by hipRTC for the device's architecture and cached per
// process, so a graph structure is compiled once however often it is
// verified.  The generated kernel takes the I/O table and the image size, or
// a batch's images.
#pragma once
#include <hip/hip_runtime.h>

#include <string>

#include "gen_abi.h"
#include "hvx_desc.h"

namespace hvx {

struct GenKernel;

// Waves of a work-group of a streamed kernel that reduces global operators:
// they share one histogram and one slot of partial results.
constexpr int kStreamRedWaves = 8;

// Launch shape of a generated kernel.
enum GenForm : int32_t {
  GEN_POINTS = 1,  // point operators only: four pixels of one row per thread, no LDS
  GEN_TILES = 2,   // LDS tiles with halos: what GEN_STREAM does not cover, one work-group per tile
  GEN_STREAM = 3,  // a wave streams a strip of columns down a band of rows, values in registers
};

// Whether a program is run by a generated kernel: everything except the
// single operators that the interpreter's own one-operator kernels already
// run with constant operators (a built-in point operator; a built-in local
// operator on U8 or F32 other than Convolve and NonLinearFilter, whose masks
// that kernel reads at run time).
bool gen_wanted(const GProg& P);

// The kernel of program P: with an output tile of tw x th, or, where they are
// 0, streamed if P allows it, else with the largest tile that fits the LDS
// budget.  Bit i of `stream` marks value i as an output that no later kernel
// reads (written with non-temporal stores).  Kernels are kept per process by
// what their source depends on: the program without its image size, the tile
// and `stream`.  Null, with the reason or the compiler's log, if P cannot be
// generated at that tile.  Compiling needs no device.
const GenKernel* gen_kernel(const GProg& P, int tw, int th, uint32_t stream, std::string* why);

// Tile of a generated kernel, or the columns of a strip and the number its
// bands' rows are a multiple of (0 x 0 for the point form).
void gen_tile(const GenKernel* k, int* tw, int* th);

// Load the kernel's code object on the current device (once per device).
hipError_t gen_load(const GenKernel* k, int device);

// Launch on stream s (gen_load must have succeeded on the current device).
// A kernel that reduces global operators (not gen_batchable) writes one slot
// of red_slot_words(P) words per work-group, gen_slots of them, to `ws`.
hipError_t gen_launch(const GenKernel* k, int device, const GProg& P, const IOTable& io, int num_cus,
                      hipStream_t s, uint32_t* ws);

// Strips of an image of the given width, and the rows of a band of a w x h
// image where one launch runs strips of the given total height (0 for the
// other forms); whole_heights: every image's height is a multiple of 4.
int gen_strips(const GenKernel* k, int w);
int gen_rows(const GenKernel* k, int w, int h, long long strip_rows, bool whole_heights, int num_cus);

// Work-groups the kernel launches for one w x h image when run over a batch
// (one per tile, one per 1024 pixels of a row for the point form, one per
// strip and band of `rows` rows for the streaming form).
long long gen_blocks(const GenKernel* k, int w, int h, int rows);

// Work-groups of gen_launch for a w x h image.
long long gen_slots(const GenKernel* k, int w, int h, int num_cus);

// Whether one launch can run the kernel over a batch of images (a kernel
// that reduces global operators cannot: each image has its own result).
bool gen_batchable(const GenKernel* k);

// One launch over n images: `imgs` in device memory, image i's work-groups
// starting at imgs[i].block0, `blocks` in all.
hipError_t gen_launch_batch(const GenKernel* k, int device, const GenBatchImage* imgs, int n, long long blocks,
                            hipStream_t s);

}  // namespace hvx
