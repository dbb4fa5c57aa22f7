// Device-side pass programs: the plain-old-data records the planner writes
// and the kernels read.  Shared between host (planner/runtime) and device
// (kernels) translation units of libqops.
#pragma once
#include <stdint.h>

namespace qops {

// Operation types inside a tile pass.
enum OpType : int32_t {
    OP_NONE = 0,
    OP_DENSE_LDS = 7, // 2^k x 2^k on tile positions, vector ALU, in LDS   a = k, pos = tile positions
    OP_MFMA = 8,      // 2^k x 2^k on tile positions, matrix cores, in LDS  a = k, pos = tile positions
    OP_DIAG_LDS = 9   // diagonal table on tile positions, in LDS (whole-state kernel)
};
// OP_MFMA / OP_DIAG_LDS / OP_DENSE_LDS in an LDS tile pass: b = 1 means `coef` is an offset
// into the coefficients staged in LDS, b = 0 (the block kept in registers, and the other
// kernels) an offset into global memory.
// OP_MFMA: c_reg (unused by LDS ops otherwise) holds QOPS_MFMA_WIDE when the
// block runs in the 32x32x2 three-product form (5-qubit blocks on the
// largest complex64 tile); its coefficients then follow that layout.
#define QOPS_MFMA_WIDE 1u

// Encoded source of one bit of a diagonal's table index (OP_DIAG_LDS pos[i]; register tiles: enc_bit).
enum BitSrc : int32_t { SRC_LANE = 0, SRC_WAVE = 1, SRC_REG = 2, SRC_GLOB = 3 };
__host__ __device__ inline int32_t enc_src(int32_t cls, int32_t v) { return (cls << 8) | v; }

// Source of a table index bit in a register tile pass, 13 bits: bit t of the
// thread number (t | 32) or bit g of the tile's base index (g << 6 | 4096), so
// that one expression reads either; 0: the bit is 0.
__host__ __device__ inline int32_t enc_bit(int32_t cls, int32_t v)
{
    return cls == SRC_LANE ? v | 32 : cls == SRC_WAVE ? (6 + v) | 32 : cls == SRC_GLOB ? v << 6 | 4096 : 0;
}

struct DevOp {              // 64 bytes
    int32_t type;
    int32_t a;
    int32_t coef;           // offset of the coefficients in the coefficient array (scalar units)
    int32_t b;
    uint32_t c_lane;        // OP_MFMA: column positions (c_lane, c_wave)
    uint32_t c_wave;
    uint32_t c_reg;
    uint32_t c_tile;        // controls on tile positions
    uint64_t c_glob;        // controls on physical bits outside the tile (checked per tile)
    int32_t pos[6];
};
static_assert(sizeof(DevOp) == 64, "DevOp layout");

// Operations of register tile passes.  One flat code selects the unrolled
// body (operation, register or lane bit, form, coefficient type), so the
// kernel branches once per operation, and the record carries its own
// coefficients, so the next one can be fetched as a whole while the current
// one runs.  complex64 records take 64 bytes, complex128 ones 128 (the second
// half of a full matrix in `more`); both live in the plan's DevOp array.
//
// A 2x2 whose bit is next targeted by another uncontrolled 2x2 runs in a
// two-coefficient form (k: w, v) that leaves a diagonal factor on the bit, and
// for register bits possibly exchanged slots; the planner folds the factor
// into that next 2x2.  Register bits with exchanged slots ("flipped": slot bit
// = 1 - bit) are resolved in the operations that read the slot index:
// register controls hold where slot & c_reg == c_val, RC_DIAG starts its table
// index at (aux >> 8) & 63, RC_REMAP carries the flipped register bits in c_reg, the
// store in PassHdr::flip.
//
// A condition on register bits is uniform per slot, and testing it at run time
// turns into compares and selects for every slot; so the common ones (one or
// two register bits, each required 1 or 0) have bodies of their own, and only
// the rest tests c_reg / c_val.  Pair (b, c), b < c, has number
// c (c - 1) / 2 + b.
enum RegCode : int32_t {
    RC_NOP = 0,            // also pads the program by one record
    RC_REMAP = 1,          // registers -> LDS -> registers        aux = new mapping
    RC_1Q_LANE = 5,        // full 2x2 on lane bit aux; + 1: controls outside the registers, + 2: any controls
    RC_X_REG = 8,          // + 3 register bit; + 1, + 2 as above
    RC_1Q_REG = 23,        // + 3 register bit; + 1, + 2 as above
    RC_SHEAR_REG = 38,     // + 6 register bit + 3 form + type (0 complex, 1 real, 2 imaginary)
    RC_SHEAR_LANE = 68,    // + 6 lane bit (0..3) + 3 exchanged + type
    RC_SHEAR_ROW = 92,     // + 12 (lane bit - 4) + 6 exchanged + 3 form + type; exchanged ones leave
                           //   the slots of register bit 0 exchanged
    // diagonal tables of 3 to 6 bits, coef: table, pos: sources (enc_bit) of
    // its index bits; aux = m | first index << 8 | index bits of the register
    // bits << 16 (3 bits each); RC_DIAG: ctl = index masks of register bits
    // 0..3 (8 bits each)
    RC_DIAG = 116,         // any register bits
    RC_DIAG0 = 117,        // none
    RC_DIAG1 = 118,        // + register bit
    RC_DIAG2 = 123,        // + pair number
    // phase k[0] (sign: -1) where every masked bit is 1
    RC_PHASE = 133,        // any register bits
    RC_PHASE0 = 134,       // none
    RC_PHASE1 = 135,       // + 2 register bit + required slot value
    RC_PHASE2 = 145,       // + 4 pair number + required slot values (bit 0: lower register bit)
    RC_SIGN = 185,         // as RC_PHASE
    RC_SIGN0 = 186,
    RC_SIGN1 = 187,
    RC_SIGN2 = 197,
    RC_CX_REG = 237,       // X on a register bit where another holds a value (no other control):
                           // + 2 (2 pair number + (1: the target is the higher one)) + required value
    // diagonal tables of at most 2 bits, entries k[0..3] by (bit 1, bit 0);
    // aux: sources of the bits that are no register bits, bit 1's << 13
    RC_TAB0 = 277,         // no register bit
    RC_TAB1 = 278,         // + register bit, which is bit 1
    RC_TAB2 = 283,         // + pair number, the lower register bit is bit 0
    RC_X_LANE = 293,       // exact X, + 3 lane bit; + 1, + 2 as RC_1Q_LANE
    RC_COUNT = 311
};

template <typename T>
struct RegOpT;
template <>
struct RegOpT<float> {
    int32_t code;
    uint32_t ctl;           // c_lane | c_wave << 8 | c_reg << 16 | c_val << 24
    int32_t coef;           // RC_DIAG: offset of the table in the coefficient array
    int32_t aux;
    uint64_t c_glob;        // controls on physical bits outside the tile (checked per tile)
    union {
        float k[8];
        int32_t pos[6];
    };
    int32_t pad[2];
};
template <>
struct RegOpT<double> {
    int32_t code;
    uint32_t ctl;
    int32_t coef;
    int32_t aux;
    uint64_t c_glob;
    union {
        double k[4];
        int32_t pos[6];
    };
    int64_t pad;
    double more[4];         // k[4..7]
    double pad2[4];
};
static_assert(sizeof(RegOpT<float>) == 64 && sizeof(RegOpT<double>) == 128, "RegOp layout");

#define QOPS_MAX_UP 10
// LDS tile passes hold physical bits 0..3 contiguously (128-byte runs of
// complex64) and choose every other tile bit; register tile passes hold bits
// 0..5 in the lanes of a wave.
#define QOPS_LDS_FIXED_BITS 4
// LDS of one work-group of the LDS tile kernel (tile plus staged
// coefficients): complex64 runs two work-groups per CU, complex128 one.
#define QOPS_LDS_TILE_BYTES_C64 (80 * 1024)
#define QOPS_LDS_TILE_BYTES_C128 (160 * 1024)
#define QOPS_MAX_QUBITS_DEV 34
#define QOPS_MAX_RUNS 12

// Header of one tile pass.  The tile holds 2^L amplitudes: tile positions
// 0..F-1 are physical bits 0..F-1 and tile position F+u is physical bit
// up_phys[u], with F = 6 for register tile passes (one lane bit each) and
// F = QOPS_LDS_FIXED_BITS for LDS tile passes.  The other physical bits
// index the tile.
struct PassHdr {
    int32_t n;
    int32_t L;
    int32_t nup;                    // L - F
    int32_t nops;
    int32_t op0;                    // first op in the op array
    uint32_t map0;                  // mapping used for the load
    int32_t nruns;                  // runs of non-tile physical bits
    int32_t lds_bytes;              // LDS the pass needs (0 if no LDS op)
    int32_t coef_src;               // LDS tile pass: coefficients staged into LDS once per
    int32_t coef_n;                 //   work-group: coef[coef_src .. coef_src + coef_n)
    int32_t up_phys[QOPS_MAX_UP];
    int32_t run_start[QOPS_MAX_RUNS];  // physical start bit of each run
    int32_t run_len[QOPS_MAX_RUNS];
    int32_t run_gshift[QOPS_MAX_RUNS]; // bit offset of the run inside the tile number
    int32_t hoist;                  // LDS tile pass: op (relative to op0) whose matrix-core
                                    //   fragments stay in registers, or -1
    int32_t flip;                   // register tile pass: register bits stored with exchanged slots
    double scale;                   // register tile pass: factor on every stored amplitude
};

// Batched executor records.
struct BatchCirc {
    void* state;        // circuits run in tile passes: their state buffer
    int32_t n;
    int32_t npass;      // tile passes
    int32_t hdr0;       // first pass header in the batch's header array
    int32_t out0;       // offset of the circuit's n <Z> outputs
    int32_t op0;        // whole-state circuits: their operations
    int32_t nops;
    int32_t part0;      // first partial-sum record of the <Z> reduction
    int32_t pad;
};
struct BatchItem {
    int32_t c;          // circuit
    int32_t tile;       // tile (pass kernels) or chunk (reduction)
};

// A mapping assigns the upper tile positions to register bits (first R
// nibbles) and wave bits (next W nibbles).
__host__ __device__ inline int32_t map_get(uint32_t m, int i) { return (int32_t)((m >> (4 * i)) & 15u); }

}  // namespace qops
