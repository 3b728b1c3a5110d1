// Compiled, never run: the form of requantisation that each window and smallest shift takes.
#include "prom.h"
#include "prom_device.h"

using namespace prom;

// plain layers: only a shift of 0 needs the general form
static_assert(pair_form_of(false, true, true, 0, 127) == kPairRelu);
static_assert(pair_form_of(false, true, false, 0, 127) == kPairLow);
static_assert(pair_form_of(false, true, true, -128, 127) == kPairFull);
static_assert(pair_form_of(false, true, false, -128, 127) == kPairFull);
static_assert(pair_form_of(false, true, true, 0, 100) == kPairClamp);
static_assert(pair_form_of(false, true, false, -100, 99) == kPairClamp);
static_assert(pair_form_of(false, true, true, 1, 127) == kPairClamp);
static_assert(pair_form_of(false, true, true, -128, 126) == kPairClamp);
static_assert(pair_form_of(false, false, false, 0, 127) == kPairAny);
static_assert(pair_form_of(false, false, false, -128, 127) == kPairAny);
static_assert(pair_form_of(false, false, false, 0, 100) == kPairAny);
// PReLU layers
static_assert(pair_form_of(true, true, true, -128, 127) == kPairPreluFull);
static_assert(pair_form_of(true, true, false, -128, 127) == kPairPreluAny);
static_assert(pair_form_of(true, true, true, -90, 127) == kPairPreluAny);
// what the shifts are reduced by in the parameters
static_assert(pair_shift_less(kPairRelu) == 2 && pair_shift_less(kPairPreluFull) == 2);
static_assert(pair_shift_less(kPairFull) == 1 && pair_shift_less(kPairLow) == 1 && pair_shift_less(kPairClamp) == 1);
static_assert(pair_shift_less(kPairAny) == 0 && pair_shift_less(kPairPreluAny) == 0);
